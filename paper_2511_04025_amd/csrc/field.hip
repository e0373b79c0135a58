// Steps 1-2 of the path: the periodic charge field of Eq. (6) on the voxel
// centers, the distance and occupancy of Eq. (7), the thickness rule, the
// element moduli E_e and the Jacobi diagonal.
//
// Field evaluation is the exact regrouping of Eq. (6): expanding
//   cos 2 pi h (x - x_j) = cos 2 pi h x cos 2 pi h x_j + sin 2 pi h x sin 2 pi h x_j
// in all three axes turns the charge sum into a tensor of (2K+1)^3 real
// coefficients over the 1D basis {1, cos 2 pi h s, sin 2 pi h s}, which is
// contracted with the basis values of each z plane (a (2K+1)^2 plane tensor),
// then of each row y, then of each voxel x.  FP64 throughout, so the hard
// threshold decides voxel for voxel like the FP64 oracle.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace shh {

// basis index u: 0 -> 1; 2h-1 -> cos(2 pi h s); 2h -> sin(2 pi h s)
__device__ __forceinline__ int basis_h(int u) { return (u + 1) >> 1; }

// ---- trig coefficient tensor of the field -----------------------------------
// one wave per coefficient, the lanes over the charges (one thread per
// coefficient walking the charges took 34 us at 48 charges: a handful of
// waves, each a chain of sincospi calls)
__global__ __launch_bounds__(256) void coef_kernel(SlotDev *s) {
  const int K = s->K, nb = s->nb, N = s->N, K1 = K + 1;
  const int e = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (e >= nb * nb * nb) return;
  const int u = e / (nb * nb), v = (e / nb) % nb, w = e % nb;
  const int h = basis_h(u), k = basis_h(v), l = basis_h(w);
  double out = 0.0;
  if (h + k + l > 0) {
    const int zeros = (h == 0) + (k == 0) + (l == 0);
    const double wgt = zeros == 0 ? 1.0 : (zeros == 1 ? 0.5 : 0.25);
    const double a = s->alpha ? s->alpha[(h * K1 + k) * K1 + l] : 1.0;
    const double c = a * wgt / double(h * h + k * k + l * l);
    double acc = 0.0;
    for (int j = lane; j < N; j += 64) {
      const double *ch = s->charges + 4 * j;
      double tx = 1.0, ty = 1.0, tz = 1.0, sn, cs;
      if (u > 0) { sincospi(2.0 * h * ch[0], &sn, &cs); tx = (u & 1) ? cs : sn; }
      if (v > 0) { sincospi(2.0 * k * ch[1], &sn, &cs); ty = (v & 1) ? cs : sn; }
      if (w > 0) { sincospi(2.0 * l * ch[2], &sn, &cs); tz = (w & 1) ? cs : sn; }
      acc += ch[3] * tx * ty * tz;
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    out = c * acc;
  }
  if (lane == 0) s->coef[e] = out;
}

// basis value and derivative at voxel center (i + 1/2)/n
__device__ __forceinline__ void basis_at(int u, int i, int n, double &val, double &der) {
  if (u == 0) { val = 1.0; der = 0.0; return; }
  const int h = basis_h(u);
  double sn, cs;
  sincospi(double(h) * double(2 * i + 1) / double(n), &sn, &cs);
  const double w = 2.0 * M_PI * h;
  if (u & 1) { val = cs; der = -w * sn; } else { val = sn; der = w * cs; }
}

// Tables of the field synthesis, in the slot's reduction scratch: the 1D basis
// at the voxel centers (values, derivatives: [n][nb] each, the same on every
// axis) and per z plane the plane tensors P[u][v] = sum_w coef[u][v][w] Z_w(z)
// and Pz (with Z_w'): [n][2][nb^2].  One workgroup per plane.  (Formed by every
// workgroup of the synthesis before, with 820 sincospi per 256 voxels.)
__host__ __device__ inline long long field_table_doubles(int n, int nb) {
  return (long long)n * (2 * nb + 2 * nb * nb);
}

__global__ __launch_bounds__(64) void field_tables_kernel(SlotDev *s) {
  __shared__ double zv[MAXB], zd[MAXB];
  const int n = s->n, nb = s->nb, z = blockIdx.x;
  double *val = s->partials, *der = val + n * nb, *planes = der + n * nb + (long long)z * 2 * nb * nb;
  for (int u = threadIdx.x; u < nb; u += 64) {
    double v, d;
    basis_at(u, z, n, v, d);
    zv[u] = val[z * nb + u] = v;
    zd[u] = der[z * nb + u] = d;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < nb * nb; e += 64) {
    double a = 0.0, b = 0.0;
    for (int w = 0; w < nb; ++w) {
      const double c = s->coef[e * nb + w];
      a += c * zv[w];
      b += c * zd[w];
    }
    planes[e] = a;
    planes[nb * nb + e] = b;
  }
}

// ---- field + gradient: 64 x FIELD_ROWS voxels of one z plane per workgroup ---
// The row tensors (sum over v, three per u) are formed once per row in LDS; a
// voxel then takes 4 NB multiply-adds.  Bound by its 32 B of output per voxel:
// 23 us at 128^3 (every voxel summed over v itself before: 114 us).
constexpr int FIELD_ROWS = 16;
template <int NB>
__global__ __launch_bounds__(256) void field_kernel(SlotDev *s) {
  __shared__ double R[FIELD_ROWS][3][NB];
  __shared__ double red[4];
  const int n = s->n;
  const int x = blockIdx.x * 64 + (threadIdx.x & 63), y0 = blockIdx.y * FIELD_ROWS, z = blockIdx.z;
  const int wave = threadIdx.x >> 6;
  const double *val = s->partials, *der = val + n * NB, *P = der + n * NB + (long long)z * 2 * NB * NB;
  for (int e = threadIdx.x; e < FIELD_ROWS * NB; e += 256) {
    const int j = e / NB, u = e % NB, y = min(y0 + j, n - 1);
    double t = 0.0, ty = 0.0, tz = 0.0;
    for (int v = 0; v < NB; ++v) {
      const double Yv = val[y * NB + v], pv = P[u * NB + v];
      t += pv * Yv;
      ty += pv * der[y * NB + v];
      tz += P[NB * NB + u * NB + v] * Yv;
    }
    R[j][0][u] = t;
    R[j][1][u] = ty;
    R[j][2][u] = tz;
  }
  const int xc = min(x, n - 1);
  double Xv[NB], Xd[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    Xv[u] = val[xc * NB + u];
    Xd[u] = der[xc * NB + u];
  }
  __syncthreads();
  const long long nn = s->nn;
  double *oF = s->F, *oG = s->G;
  double gn = 0.0;
  for (int j = wave; j < FIELD_ROWS; j += 4) {
    const int y = y0 + j;
    if (x >= n || y >= n) break;
    double F = 0.0, Gx = 0.0, Gy = 0.0, Gz = 0.0;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      F += Xv[u] * R[j][0][u];
      Gx += Xd[u] * R[j][0][u];
      Gy += Xv[u] * R[j][1][u];
      Gz += Xv[u] * R[j][2][u];
    }
    const long long idx = ((long long)z * n + y) * n + x;
    oF[idx] = F;
    oG[idx] = Gx;
    oG[nn + idx] = Gy;
    oG[2 * nn + idx] = Gz;
    gn = fmax(gn, sqrt(Gx * Gx + Gy * Gy + Gz * Gz));
  }
  // workgroup max, then a bitwise atomic max (non-negative doubles order as integers)
  for (int off = 32; off > 0; off >>= 1) gn = fmax(gn, __shfl_xor(gn, off, 64));
  if ((threadIdx.x & 63) == 0) red[wave] = gn;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    atomicMax(&s->st->gmax_bits, (unsigned long long)__double_as_longlong(m));
  }
}

// ---- hard step: bins of the order-statistic search (below) -------------------
constexpr int SEL_BITS = 11, SEL_BINS = 1 << SEL_BITS, SEL_PASSES = 6;  // 6 x 11 >= 64
constexpr int SEL_T = 512;   // threads of a counting workgroup
constexpr unsigned long long INF_BITS = 0x7FF0000000000000ull;

// ---- distance d = |F - c| / max(||grad F||, 1e-12 max ||grad F||) ------------
__global__ __launch_bounds__(256) void distance_kernel(SlotDev *s) {
  const long long nn = s->nn;
  // the order-statistic search that may follow counts into zeroed bins (the
  // tables of the synthesis were here)
  const long long first = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long long i = first; i < 2 * SEL_BINS * SEL_PASSES; i += (long long)gridDim.x * blockDim.x) ((unsigned *)s->partials)[i] = 0u;
  const double gmax = __longlong_as_double((long long)s->st->gmax_bits);
  const double gmin = 1e-12 * gmax;
  const int mode = s->dist_mode;
  const double iso = s->iso;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nn;
       i += (long long)gridDim.x * blockDim.x) {
    const double num = fabs(s->F[i] - iso);
    double d;
    if (mode == 1) {
      d = num;
    } else {
      const double gx = s->G[i], gy = s->G[nn + i], gz = s->G[2 * nn + i];
      const double den = fmax(sqrt(gx * gx + gy * gy + gz * gz), gmin);
      d = num > 0.0 ? num / den : 0.0;  // 0/0 -> 0; num/0 -> +inf
    }
    s->d[i] = d;
  }
}

// ---- hard step: the k1-th and k2-th smallest distance (1-based) ---------------
// Non-negative doubles (and +inf, which a NaN counts as) order like their bit
// patterns.  A radix search from the top: pass p counts, among the elements that
// share the digits found so far, the next 11 bits (per search: the two ranks may
// part), in LDS bins that go to the pass's global bins.  The next pass finds the
// digit that holds the rank, every workgroup for itself: with a last-arrival step
// (a release per workgroup, one workgroup's scan) a pass took 17 us at 128^3
// instead of 8.  (A 16-way search by counting against 15 pivots per rank took 18
// launches of 32 us.)
struct SelState {  // at the entry of a pass
  unsigned long long pre[2];   // the digits found
  unsigned long long rank[2];  // the rank left below them
};
__device__ __forceinline__ unsigned *sel_bins(SlotDev *s, int pass) {
  return (unsigned *)s->partials + pass * 2 * SEL_BINS;
}
__device__ __forceinline__ SelState *sel_state(SlotDev *s, int pass) {
  return (SelState *)((unsigned *)s->partials + SEL_PASSES * 2 * SEL_BINS) + pass;
}

// the state at the entry of `pass` (> 0) from that of the pass before and its
// counts; all threads of a SEL_T workgroup
__device__ __forceinline__ void sel_advance(SlotDev *s, int pass, SelState &out, SelState *shared_state,
                                            unsigned (*wave_sum)[SEL_T / 64]) {
  constexpr int PER = SEL_BINS / SEL_T;
  const SelState in = *sel_state(s, pass - 1);
  const unsigned *g = sel_bins(s, pass - 1);
  const int shift = SEL_BITS * (SEL_PASSES - pass);
  const bool same = in.pre[0] == in.pre[1];  // one count serves both
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned c[2][PER], below[2];  // thread t owns bins [PER t, PER t + PER) of each search
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    unsigned sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      c[j][i] = g[(same ? 0 : j) * SEL_BINS + threadIdx.x * PER + i];
      sum += c[j][i];
    }
    unsigned inc = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned v = __shfl_up(inc, off, 64);
      inc += lane >= off ? v : 0u;
    }
    if (lane == 63) wave_sum[j][wave] = inc;
    below[j] = inc - sum;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    unsigned long long n = below[j];
    for (int w = 0; w < wave; ++w) n += wave_sum[j][w];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (n < in.rank[j] && in.rank[j] <= n + c[j][i]) {  // exactly one bin holds the rank
        shared_state->pre[j] = in.pre[j] | ((unsigned long long)(threadIdx.x * PER + i) << shift);
        shared_state->rank[j] = in.rank[j] - n;
      }
      n += c[j][i];
    }
  }
  __syncthreads();
  out = *shared_state;
}

__global__ __launch_bounds__(SEL_T) void select_pass_kernel(SlotDev *s, int pass, long long k1, long long k2,
                                                            int nblocks) {
  __shared__ unsigned bins[2][SEL_BINS];
  __shared__ unsigned wave_sum[2][SEL_T / 64];
  __shared__ SelState entry;
  for (int i = threadIdx.x; i < 2 * SEL_BINS; i += SEL_T) (&bins[0][0])[i] = 0u;
  SelState at = {{0ull, 0ull}, {(unsigned long long)k1, (unsigned long long)k2}};
  if (pass) sel_advance(s, pass, at, &entry, wave_sum);
  else __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x == 0) *sel_state(s, pass) = at;
  // 64 = 5 x 11 + 9: the first digit has 9 bits
  const int shift = SEL_BITS * (SEL_PASSES - 1 - pass);
  const bool same = at.pre[0] == at.pre[1];
  const long long nn = s->nn;
  const int hi = shift + SEL_BITS;  // bits above the digit (none in the first pass)
  constexpr int UN = 4;             // loads in flight per thread
  const double *d = s->d;
  const long long stride = (long long)nblocks * SEL_T;
  for (long long e0 = (long long)blockIdx.x * SEL_T + threadIdx.x; e0 < nn; e0 += UN * stride) {
    unsigned long long v[UN];
#pragma unroll
    for (int j = 0; j < UN; ++j) {
      const long long e = e0 + j * stride;
      v[j] = (unsigned long long)__double_as_longlong(d[e < nn ? e : e0]);
    }
#pragma unroll
    for (int j = 0; j < UN; ++j) {
      if (e0 + j * stride >= nn) break;
      const unsigned long long b = v[j] < INF_BITS ? v[j] : INF_BITS;
      const unsigned dig = unsigned(b >> shift) & (SEL_BINS - 1);
      const unsigned long long top = pass ? b >> hi : 0ull;
      if (top == (pass ? at.pre[0] >> hi : 0ull)) atomicAdd(&bins[0][dig], 1u);
      if (!same && top == at.pre[1] >> hi) atomicAdd(&bins[1][dig], 1u);
    }
  }
  __syncthreads();
  unsigned *g = sel_bins(s, pass);
  for (int i = threadIdx.x; i < 2 * SEL_BINS; i += SEL_T)
    if (const unsigned c = (&bins[0][0])[i]) atomicAdd(&g[i], c);
}

// t from the two order statistics; k = round(vf n^3).
__global__ __launch_bounds__(SEL_T) void select_finish_kernel(SlotDev *s, long long k) {
  __shared__ unsigned wave_sum[2][SEL_T / 64];
  __shared__ SelState entry;
  SelState at;
  sel_advance(s, SEL_PASSES, at, &entry, wave_sum);
  if (threadIdx.x != 0) return;
  const double v1 = __longlong_as_double((long long)at.pre[0]);
  const double v2 = __longlong_as_double((long long)at.pre[1]);
  double t;
  if (k <= 0) t = 0.5 * v1;                 // v1 = smallest
  else if (k >= s->nn) t = 2.0 * v2 + 1.0;  // v2 = largest
  else t = 0.5 * (v1 + v2);
  s->st->t = t;
}

// ---- logistic: bisection on t until |V(t) - target| <= 1e-12, 200 steps at most ----
// A pass evaluates the midpoints that its steps can reach (three steps, seven
// midpoints; on large grids, where a midpoint's logistics cost more than a
// launch, one) and leaves per-workgroup sums; the next one takes those steps in every workgroup
// for itself (no last-arrival step, as in the search above), from the state that
// its predecessor started from: states and sums alternate between two places.
// The steps are those of the plain bisection.  The field of a logistic design went
// from 1.55 to 0.63 ms at 96^3 and from 4.31 to 3.14 at 256^3 (200 launches of one
// step with a last-arrival sum, most of them after the end).
constexpr int BIS_T = 512, BIS_BLOCKS = 1024, BIS_STEPS = 200;
// three steps a pass up to 128^3: field with three / one at 96^3 0.63 / 0.83 ms,
// 128^3 0.95 / 0.96, 160^3 1.51 / 1.23
constexpr long long BIS_SMALL = 128LL * 128 * 128;
struct BisState {
  double lo, hi, t;
  int done, steps;
};
__device__ __forceinline__ double *bis_parts(SlotDev *s, int pass) { return s->partials + (pass & 1) * BIS_BLOCKS * 8; }
__device__ __forceinline__ BisState *bis_state(SlotDev *s, int pass) {
  return (BisState *)(s->partials + 2 * BIS_BLOCKS * 8) + (pass & 1);
}

// node i of the tree of midpoints; its lower and upper half continue at 2 i + 1, 2 i + 2
template <int NODES>
__device__ __forceinline__ void bis_nodes(const BisState &b, double (&t)[NODES]) {
  double lo[NODES], hi[NODES];
  lo[0] = b.lo;
  hi[0] = b.hi;
#pragma unroll
  for (int i = 0; i < NODES; ++i) {
    t[i] = 0.5 * (lo[i] + hi[i]);
    if (2 * i + 2 < NODES) {
      lo[2 * i + 1] = lo[i];
      hi[2 * i + 1] = t[i];
      lo[2 * i + 2] = t[i];
      hi[2 * i + 2] = hi[i];
    }
  }
}

__device__ __forceinline__ double logistic(double kappa, double t, double d) {
  // 1 / (1 + exp(-kappa (t - d))), stable for both signs
  const double a = kappa * (t - d);
  if (a >= 0.0) return 1.0 / (1.0 + exp(-a));
  const double e = exp(a);
  return e / (1.0 + e);
}

// min and max of d by workgroup, as bit patterns (non-negative doubles order like
// them, +inf and a NaN last)
__device__ __forceinline__ void wave_minmax(unsigned long long &mn, unsigned long long &mx) {
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long a = __shfl_xor(mn, off, 64), b = __shfl_xor(mx, off, 64);
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
  }
}

__global__ __launch_bounds__(BIS_T) void minmax_d_kernel(SlotDev *s, int nblocks) {
  __shared__ unsigned long long red[2][BIS_T / 64];
  const long long nn = s->nn;
  unsigned long long mn = ~0ull, mx = 0ull;
  for (long long i = (long long)blockIdx.x * BIS_T + threadIdx.x; i < nn; i += (long long)nblocks * BIS_T) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(s->d[i]);
    mn = b < mn ? b : mn;
    mx = b > mx ? b : mx;
  }
  wave_minmax(mn, mx);
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = mn;
    red[1][threadIdx.x >> 6] = mx;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < BIS_T / 64; ++w) {
    mn = red[0][w] < mn ? red[0][w] : mn;
    mx = red[1][w] > mx ? red[1][w] : mx;
  }
  unsigned long long *part = (unsigned long long *)s->partials + 2 * blockIdx.x;
  part[0] = mn;
  part[1] = mx;
}

__global__ __launch_bounds__(64) void bisect_init_kernel(SlotDev *s, int nblocks) {
  const unsigned long long *part = (const unsigned long long *)s->partials;
  unsigned long long mn = ~0ull, mx = 0ull;
  for (int b = threadIdx.x; b < nblocks; b += 64) {
    mn = part[2 * b] < mn ? part[2 * b] : mn;
    mx = part[2 * b + 1] > mx ? part[2 * b + 1] : mx;
  }
  wave_minmax(mn, mx);
  if (threadIdx.x != 0) return;
  BisState b;
  b.lo = __longlong_as_double((long long)mn) - 40.0 / s->kappa;
  b.hi = __longlong_as_double((long long)mx) + 40.0 / s->kappa;
  b.t = 0.5 * (b.lo + b.hi);
  b.done = 0;
  b.steps = 0;
  *bis_state(s, 0) = b;
}

// the state at the entry of pass > 0: its steps from that of the pass
// before with its sums; all threads of a BIS_T workgroup
template <int LEVELS>
__device__ __forceinline__ BisState bis_advance(SlotDev *s, int pass, int nblocks, double *red, BisState *shared_state) {
  constexpr int NODES = (1 << LEVELS) - 1;
  BisState b = *bis_state(s, pass - 1);
  if (b.done) return b;  // uniform
  double t[NODES], tot[NODES];
  bis_nodes<NODES>(b, t);
  sum_partials<NODES, 8>(bis_parts(s, pass - 1), nblocks, tot, red, BIS_T);
  if (threadIdx.x == 0) {
    const double n = double(s->nn), target = s->target_vf;
    int at = 0;
#pragma unroll
    for (int level = 0; level < LEVELS; ++level) {
      if (b.done) continue;
      double tt = 0.0, V = 0.0;
#pragma unroll
      for (int i = 0; i < NODES; ++i)  // (no indexed registers)
        if (i == at) {
          tt = t[i];
          V = tot[i] / n;
        }
      b.t = tt;
      b.steps += 1;
      if (fabs(V - target) <= 1e-12) {
        b.done = 1;
      } else if (V < target) {
        b.lo = tt;
        at = 2 * at + 2;
      } else {
        b.hi = tt;
        at = 2 * at + 1;
      }
      if (b.steps == BIS_STEPS) b.done = 1;
    }
    *shared_state = b;
  }
  __syncthreads();
  return *shared_state;
}

template <int LEVELS>
__global__ __launch_bounds__(BIS_T) void bisect_pass_kernel(SlotDev *s, int pass, int nblocks) {
  constexpr int NODES = (1 << LEVELS) - 1;
  __shared__ double red[7 * 16];
  __shared__ BisState entry;
  BisState b;
  if (pass) {
    b = bis_advance<LEVELS>(s, pass, nblocks, red, &entry);
    if (blockIdx.x == 0 && threadIdx.x == 0) *bis_state(s, pass) = b;
  } else {
    b = *bis_state(s, 0);
  }
  if (b.done) return;
  double t[NODES], v[NODES];
  bis_nodes<NODES>(b, t);
#pragma unroll
  for (int i = 0; i < NODES; ++i) v[i] = 0.0;
  const double kappa = s->kappa;
  const long long nn = s->nn;
  for (long long e = (long long)blockIdx.x * BIS_T + threadIdx.x; e < nn; e += (long long)nblocks * BIS_T) {
    const double d = s->d[e];
#pragma unroll
    for (int i = 0; i < NODES; ++i) v[i] += logistic(kappa, t[i], d);
  }
  __syncthreads();  // the sums above have been read from red
  block_sum<NODES>(v, red, BIS_T);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < NODES; ++i) bis_parts(s, pass)[8 * blockIdx.x + i] = v[i];
  }
}

template <int LEVELS>
__global__ __launch_bounds__(BIS_T) void bisect_finish_kernel(SlotDev *s, int passes, int nblocks) {
  __shared__ double red[7 * 16];
  __shared__ BisState entry;
  const BisState b = bis_advance<LEVELS>(s, passes, nblocks, red, &entry);
  if (threadIdx.x == 0) s->st->t = b.t;
}

// ---- occupancy, element moduli and volume fraction ---------------------------
// (The sums are finished by a kernel of one workgroup: a last-arrival counter
// needs every workgroup's device-wide release, which writes the L2's dirty lines
// back.  128^3: 37 us in one kernel, 10 + 4 in two; the given moduli of 101^3 36
// and 13 + 3.)
__global__ __launch_bounds__(256) void occupancy_kernel(SlotDev *s, double *beta_out, int nblocks) {
  __shared__ double red[16];
  const CgState *st = s->st;
  const double t = st->t, kappa = s->kappa, E = s->E, Ev = s->E_void;
  const long long nn = s->nn;
  double v[1] = {0.0};  // V = mean beta over every voxel, culled or not
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nn;
       i += (long long)nblocks * blockDim.x) {
    const double d = s->d[i];
    const double b = kappa == 0.0 ? (d < t ? 1.0 : 0.0) : logistic(kappa, t, d);
    const double e = s->cull > 0.0 ? (b > s->cull ? E * b : 0.0) : Ev + (E - Ev) * b;
    s->E64[i] = e;
    if (s->E32) s->E32[i] = (float)e;
    if (beta_out) beta_out[i] = b;
    v[0] += b;
  }
  block_sum<1>(v, red, 256);
  if (threadIdx.x == 0) s->partials[4 * blockIdx.x] = v[0];
}

__global__ __launch_bounds__(256) void occupancy_sum_kernel(SlotDev *s, int nblocks) {
  __shared__ double red[16];
  double tot[1];
  sum_partials<1>(s->partials, nblocks, tot, red, 256);
  if (threadIdx.x == 0) s->st->V = tot[0] / double(s->nn);
}

// Moduli given directly (solver-only entries).  The source grid is one of
//   DT = 0: a 1-byte solid/void code, E_e = E where the code is nonzero, else E_void
//   DT = 1: float moduli,  DT = 2: double moduli.
template <int DT>
__device__ __forceinline__ double decode_modulus(const void *E, long long i, double Es, double Ev) {
  if constexpr (DT == 0) return ((const unsigned char *)E)[i] ? Es : Ev;
  else if constexpr (DT == 1) return (double)((const float *)E)[i];
  else return ((const double *)E)[i];
}

// ---- inverse Jacobi diagonal: ((lambda + 4 mu)/9 * sum of the 8 incident E_e)^-1 --
template <typename T>
__global__ __launch_bounds__(256) void dinv_kernel(SlotDev *s) {
  const int n = s->n;
  const long long nn = s->nn;
  const double c = (s->lam + 4.0 * s->mu) / 9.0;
  T *Dinv = (T *)s->Dinv;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nn;
       i += (long long)gridDim.x * blockDim.x) {
    const int x = int(i % n), y = int((i / n) % n), z = int(i / ((long long)n * n));
    const int xm = x == 0 ? n - 1 : x - 1, ym = y == 0 ? n - 1 : y - 1, zm = z == 0 ? n - 1 : z - 1;
    const double *E = s->E64;
    auto at = [&](int a, int b, int cc) { return E[((long long)cc * n + b) * n + a]; };
    const double sum = ((at(x, y, z) + at(xm, y, z)) + (at(x, ym, z) + at(xm, ym, z))) +
                       ((at(x, y, zm) + at(xm, y, zm)) + (at(x, ym, zm) + at(xm, ym, zm)));
    const double dg = c * sum;
    Dinv[i] = (T)(dg > 0.0 ? 1.0 / dg : 0.0);
  }
}

// Moduli given directly: copy, round, the Jacobi diagonal (from the source grid)
// and the volume fraction -- the solid share of the code (DT = 0), else mean(E)
// / max(E) -- in one pass.  (The maximum by 4,096 atomics on one word, the copy
// and the diagonal one after another took 87 us at 101^3.)
template <int DT, typename T>
__global__ __launch_bounds__(256) void moduli_kernel(SlotDev *s, const void *E, double Es, double Ev, int nblocks) {
  __shared__ double red[16];
  const int n = s->n;
  const long long nn = s->nn;
  const double cd = (s->lam + 4.0 * s->mu) / 9.0;
  double *oE = s->E64;
  float *oE32 = s->E32;
  T *Dinv = (T *)s->Dinv;
  double v[1] = {0.0}, mx = 0.0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nn;
       i += (long long)nblocks * blockDim.x) {
    const unsigned row = unsigned(i) / unsigned(n);  // n <= 512: node indices fit 32 bits
    const int x = int(unsigned(i) - row * unsigned(n)), y = int(row % unsigned(n)), z = int(row / unsigned(n));
    const int xm = x == 0 ? n - 1 : x - 1, ym = y == 0 ? n - 1 : y - 1, zm = z == 0 ? n - 1 : z - 1;
    auto at = [&](int a, int b, int c) { return decode_modulus<DT>(E, ((long long)c * n + b) * n + a, Es, Ev); };
    const double e = at(x, y, z);
    const double sum = ((e + at(xm, y, z)) + (at(x, ym, z) + at(xm, ym, z))) +
                       ((at(x, y, zm) + at(xm, y, zm)) + (at(x, ym, zm) + at(xm, ym, zm)));
    oE[i] = e;
    if (oE32) oE32[i] = (float)e;
    const double dg = cd * sum;
    Dinv[i] = (T)(dg > 0.0 ? 1.0 / dg : 0.0);
    if constexpr (DT == 0) v[0] += ((const unsigned char *)E)[i] ? 1.0 : 0.0;
    else v[0] += e;
    mx = e > mx ? e : mx;  // a NaN or negative modulus never counts
  }
  block_sum<1>(v, red, 256);
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    s->partials[4 * blockIdx.x] = v[0];
    s->partials[4 * blockIdx.x + 1] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  }
}

// maximum and volume fraction from the workgroups' partials (see the occupancy)
template <int DT>
__global__ __launch_bounds__(256) void moduli_sum_kernel(SlotDev *s, int nblocks) {
  __shared__ double red[16];
  CgState *st = s->st;
  const long long nn = s->nn;
  double tot[1];
  sum_partials<1>(s->partials, nblocks, tot, red, 256);
  double m = 0.0;
  for (int k = threadIdx.x; k < nblocks; k += 256) m = fmax(m, s->partials[4 * k + 1]);
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double emax = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    st->Emax = emax;
    if constexpr (DT == 0) st->V = tot[0] / double(nn);
    else st->V = emax > 0.0 ? tot[0] / double(nn) / emax : 0.0;
    st->t = 0.0;
  }
}

// ---- host launchers ------------------------------------------------------------
static int grid_for(long long nn, int cap) {
  long long g = (nn + 255) / 256;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return int(g);
}

hipError_t launch_coef(SlotDev *d_slot, int nb, hipStream_t st) {
  coef_kernel<<<(nb * nb * nb + 3) / 4, 256, 0, st>>>(d_slot);
  return hipGetLastError();
}

// scratch: doubles in the slot's reduction scratch
hipError_t launch_field(SlotDev *d_slot, int n, int nb, long long scratch, hipStream_t st) {
  if (scratch < field_table_doubles(n, nb)) return hipErrorInvalidValue;
  hipError_t rc = launch_coef(d_slot, nb, st);
  if (rc != hipSuccess) return rc;
  field_tables_kernel<<<n, 64, 0, st>>>(d_slot);
  const dim3 g((n + 63) / 64, (n + FIELD_ROWS - 1) / FIELD_ROWS, n);
  switch (nb) {
    case 3: field_kernel<3><<<g, 256, 0, st>>>(d_slot); break;
    case 5: field_kernel<5><<<g, 256, 0, st>>>(d_slot); break;
    case 7: field_kernel<7><<<g, 256, 0, st>>>(d_slot); break;
    case 9: field_kernel<9><<<g, 256, 0, st>>>(d_slot); break;
    case 11: field_kernel<11><<<g, 256, 0, st>>>(d_slot); break;
    case 13: field_kernel<13><<<g, 256, 0, st>>>(d_slot); break;
    default: return hipErrorInvalidValue;  // K is 1 to MAXK
  }
  const long long nn = (long long)n * n * n;
  distance_kernel<<<grid_for(nn, 8192), 256, 0, st>>>(d_slot);
  return hipGetLastError();
}

int reduce_blocks(long long nn) { return grid_for(nn, 1024); }

hipError_t launch_select_hard(SlotDev *d_slot, long long nn, long long k, hipStream_t st) {
  // one workgroup per CU at most, 16 elements per thread at least: every
  // workgroup adds its bins to the global ones
  const int nbk = (int)std::max(1LL, std::min(256LL, (nn + 4095) / 4096));
  const long long k1 = k <= 0 ? 1 : (k >= nn ? nn : k);
  const long long k2 = k <= 0 ? 1 : (k >= nn ? nn : k + 1);
  for (int p = 0; p < SEL_PASSES; ++p) select_pass_kernel<<<nbk, SEL_T, 0, st>>>(d_slot, p, k1, k2, nbk);
  select_finish_kernel<<<1, SEL_T, 0, st>>>(d_slot, k);
  return hipGetLastError();
}

template <int LEVELS>
static void launch_bisect_levels(SlotDev *d_slot, int nbk, hipStream_t st) {
  constexpr int passes = (BIS_STEPS + LEVELS - 1) / LEVELS;
  minmax_d_kernel<<<nbk, BIS_T, 0, st>>>(d_slot, nbk);
  bisect_init_kernel<<<1, 64, 0, st>>>(d_slot, nbk);
  for (int p = 0; p < passes; ++p) bisect_pass_kernel<LEVELS><<<nbk, BIS_T, 0, st>>>(d_slot, p, nbk);
  bisect_finish_kernel<LEVELS><<<1, BIS_T, 0, st>>>(d_slot, passes, nbk);
}

hipError_t launch_bisect(SlotDev *d_slot, long long nn, hipStream_t st) {
  const long long g = (nn + BIS_T - 1) / BIS_T;
  if (nn <= BIS_SMALL) launch_bisect_levels<3>(d_slot, (int)std::max(1LL, std::min(256LL, g)), st);
  else launch_bisect_levels<1>(d_slot, (int)std::min((long long)BIS_BLOCKS, g), st);
  return hipGetLastError();
}

hipError_t launch_occupancy(SlotDev *d_slot, long long nn, double *beta_out, hipStream_t st) {
  const int nbk = reduce_blocks(nn);
  occupancy_kernel<<<nbk, 256, 0, st>>>(d_slot, beta_out, nbk);
  occupancy_sum_kernel<<<1, 256, 0, st>>>(d_slot, nbk);
  return hipGetLastError();
}

hipError_t launch_moduli(SlotDev *d_slot, long long nn, const void *E, int e_dtype, double Es, double Ev, int prec,
                         hipStream_t st) {
  const int nbk = reduce_blocks(nn);
  auto go = [&](auto dt) {
    constexpr int DT = decltype(dt)::value;
    if (prec == 0) moduli_kernel<DT, double><<<nbk, 256, 0, st>>>(d_slot, E, Es, Ev, nbk);
    else moduli_kernel<DT, float><<<nbk, 256, 0, st>>>(d_slot, E, Es, Ev, nbk);
    moduli_sum_kernel<DT><<<1, 256, 0, st>>>(d_slot, nbk);
  };
  if (e_dtype == 0) go(std::integral_constant<int, 0>{});
  else if (e_dtype == 1) go(std::integral_constant<int, 1>{});
  else go(std::integral_constant<int, 2>{});
  return hipGetLastError();
}

hipError_t launch_dinv(SlotDev *d_slot, long long nn, int prec, hipStream_t st) {
  if (prec == 0) dinv_kernel<double><<<grid_for(nn, 8192), 256, 0, st>>>(d_slot);
  else dinv_kernel<float><<<grid_for(nn, 8192), 256, 0, st>>>(d_slot);
  return hipGetLastError();
}

}  // namespace shh
