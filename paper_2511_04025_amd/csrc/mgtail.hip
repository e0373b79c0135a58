// The last two multigrid levels of the 3 x 2^k grids in one launch: restriction
// into the last smoothed level (6^3 nodes), its pre-smoothing, the dense solve
// on 3^3 nodes, the post-smoothing and the prolongation out of it.
//
// Why: eight launches whose work is a few microseconds of latency each took
// 30 us of a cycle (FP64: 45).  One workgroup of 16 waves holds a load case:
// each node's 14 stored stencil blocks stay in the registers of four threads
// over the four operator passes (they are read once), the vectors in LDS.  A
// pass has two halves: thread (node, group) multiplies its blocks by the
// neighbours' values and their transposes by its own value, which LDS carries
// to the neighbours; then thread (node, component) sums.  12 us (FP64: 23),
// a third of it the first loads' latency, 1 us (FP64: 3) a pass; one 48^3
// design 12.1 -> 10.5 ms, a 24^3 one in FP64 14.6 -> 11.8 ms.  In FP64 the blocks
// take 72 of the 128 registers that 1,024 threads leave, and 13 values go to
// scratch (48 bytes a thread).
// The 8^3 -> 4^3 tails of the powers of two keep their launches: there the
// blocks (258 KB) and the dense inverse (295 KB) come to one compute unit at
// 25 GB/s, 11 + 17 us, and the whole took 35 us against 45 with the launches'
// gaps on one design, no gain on a batch.
#include "kernels.hpp"
#include "mg.hpp"

namespace shh {

constexpr int TAIL_N = 6;

template <typename T>
__global__ __launch_bounds__(1024) void mg_tail_kernel(MgBatch B, int l, int fine) {
  constexpr int n = TAIL_N, nn = n * n * n, nc = n / 2, nd = 3 * nc * nc * nc;
  constexpr int NP = 256;                    // padded nodes
  constexpr int G = 1024 / NP;               // threads per node
  constexpr int KB = (MG_HALF + G - 1) / G;  // stored blocks per thread
  constexpr int CP = 1024 / nd;              // partial sums per coarsest unknown
  constexpr int CJ = (nd + CP - 1) / CP;
  static_assert(nn <= NP && G > 3, "one component of one node a thread");
  __shared__ T vec[3][NP];
  __shared__ T fwd[G][3][NP];
  __shared__ T bwd[MG_HALF - 1][3][NP];
  __shared__ T cb[nd], cx[nd];
  __shared__ double cpart[CP][nd];
  const int rhs = blockIdx.x;
  const SlotDev *s = B.slot[blockIdx.y];
  const MgDev *mg = B.mg[blockIdx.y];
  if (!s->st->active[rhs]) return;
  const MgLevel &L = mg->lv[l];
  const int v = threadIdx.x & (NP - 1), g = __builtin_amdgcn_readfirstlane(threadIdx.x / NP);
  const bool in = v < nn;
  const int vv = in ? v : 0;
  const int x = vv % n, y = (vv / n) % n, z = vv / (n * n);
  const int xm = x == 0 ? n - 1 : x - 1, xp = x + 1 == n ? 0 : x + 1;
  const int ym = y == 0 ? n - 1 : y - 1, yp = y + 1 == n ? 0 : y + 1;
  const int zm = z == 0 ? n - 1 : z - 1, zp = z + 1 == n ? 0 : z + 1;
  const T c1 = (T)L.c1, c2 = (T)L.c2, ith = (T)L.inv_theta;

  // the node's blocks g, g + G, ... and the neighbours they couple it to
  T S[KB][9];
  int nb[KB];
  {
    const SHH_GLOBAL T *Sg = to_global((const T *)L.S);
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      const int k = g + i * G;  // uniform over the wave
      const int w = 13 + k, dz = w / 9 - 1, dy = (w / 3) % 3 - 1, dx = w % 3 - 1;
      nb[i] = ((dz > 0 ? zp : z) * n + (dy < 0 ? ym : (dy > 0 ? yp : y))) * n + (dx < 0 ? xm : (dx > 0 ? xp : x));
#pragma unroll
      for (int e = 0; e < 9; ++e) S[i][e] = k < MG_HALF ? Sg[(k * 9 + e) * nn + vv] : T(0);
    }
  }
  // groups 0, 1, 2 finish component g of the node
  const bool mine = g < 3 && in;
  const int c = g < 3 ? g : 0;
  T b = T(0), dv = T(0), r, d, xx;
  if (mine) {
    dv = to_global((const T *)L.Dinv)[c * nn + vv];
    if (fine) {  // b = P^T r of the level above
      const MgLevel &F = mg->lv[l - 1];
      const int nf = F.n;
      const SHH_GLOBAL T *rf = to_global((const T *)F.r) + ((long long)rhs * 3 + c) * F.nn;
      const int fx[3] = {x == 0 ? nf - 1 : 2 * x - 1, 2 * x, 2 * x + 1};
#pragma unroll(sizeof(T) == 4 ? 3 : 1)  // FP64: no room for 27 values beside the blocks
      for (int oz = 0; oz < 3; ++oz) {
        const int Z = 2 * z + oz - 1;
        T val[3][3];
#pragma unroll
        for (int oy = 0; oy < 3; ++oy) {
          const int Y = 2 * y + oy - 1;
          const int ro = ((Z < 0 ? nf - 1 : Z) * nf + (Y < 0 ? nf - 1 : Y)) * nf;
#pragma unroll
          for (int j = 0; j < 3; ++j) val[oy][j] = rf[ro + fx[j]];
        }
        const T wz = oz != 1 ? T(0.5) : T(1);
#pragma unroll
        for (int oy = 0; oy < 3; ++oy)
          b += (oy != 1 ? T(0.5) * wz : wz) * (val[oy][1] + T(0.5) * (val[oy][2] + val[oy][0]));
      }
    } else {
      b = to_global((const T *)L.b)[(rhs * 3 + c) * nn + vv];
    }
  }
  d = dv * b * ith;
  if (g < 3) vec[g][v] = d;
  __syncthreads();

  // A vec at this thread's component
  auto apply = [&]() -> T {
    T own[3], acc[3] = {T(0), T(0), T(0)};
#pragma unroll
    for (int c = 0; c < 3; ++c) own[c] = vec[c][v];
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      const int k = g + i * G;
      T u[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) u[c] = vec[c][nb[i]];
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int j = 0; j < 3; ++j) acc[c] += S[i][3 * c + j] * u[j];
      if (k > 0 && k < MG_HALF) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          T t = T(0);
#pragma unroll
          for (int j = 0; j < 3; ++j) t += S[i][3 * j + c] * own[j];
          bwd[k - 1][c][v] = t;
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) fwd[g][c][v] = acc[c];
    __syncthreads();
    T sum = T(0);
    if (g < 3) {
#pragma unroll
      for (int h = 0; h < G; ++h) sum += fwd[h][g][v];
#pragma unroll
      for (int k = 1; k < MG_HALF; ++k) {  // the block of offset w, stored at v - w
        const int w = 13 + k, dz = w / 9 - 1, dy = (w / 3) % 3 - 1, dx = w % 3 - 1;
        const int u =
            ((dz > 0 ? zm : z) * n + (dy < 0 ? yp : (dy > 0 ? ym : y))) * n + (dx < 0 ? xp : (dx > 0 ? xm : x));
        sum += bwd[k - 1][g][u];
      }
    }
    return sum;
  };
  // the next operand; all have read this pass's when its second half runs
  auto publish = [&](T val) {
    if (g < 3) vec[g][v] = val;
    __syncthreads();
  };

  r = b - apply();
  {
    const T d1 = c1 * d + c2 * dv * r;
    xx = d + d1;
    d = d1;
  }
  publish(d);
  r -= apply();
  publish(r);
  // coarse right-hand side, the dense solve and its correction
  if (threadIdx.x < nd) {
    const int t = threadIdx.x, c = t % 3, I = t / 3;
    const int X = I % nc, Y = (I / nc) % nc, Z = I / (nc * nc);
    T a = T(0);
#pragma unroll
    for (int o = 0; o < 9; ++o) {
      const int fz = 2 * Z + o / 3 - 1, fy = 2 * Y + o % 3 - 1;
      const int ro = ((fz < 0 ? n - 1 : fz) * n + (fy < 0 ? n - 1 : fy)) * n;
      const T wyz = T((o / 3 != 1 ? 0.5 : 1.0) * (o % 3 != 1 ? 0.5 : 1.0));
      a += wyz * (vec[c][ro + 2 * X] + T(0.5) * (vec[c][ro + 2 * X + 1] + vec[c][ro + (X == 0 ? n - 1 : 2 * X - 1)]));
    }
    cb[t] = a;
  }
  __syncthreads();
  {
    // the inverse is symmetric: column `row` read as row j, coalesced
    const SHH_GLOBAL double *M = to_global((const double *)mg->Mc);
    const int p = threadIdx.x / nd, row = threadIdx.x % nd;
    if (p < CP) {
      double a = 0.0;
#pragma unroll
      for (int i = 0; i < CJ; ++i) {
        const int j = p + i * CP;
        if (j < nd) a += M[j * nd + row] * (double)cb[j];
      }
      cpart[p][row] = a;
    }
    __syncthreads();
    if (threadIdx.x < nd) {
      double t = 0.0;
#pragma unroll
      for (int h = 0; h < CP; ++h) t += cpart[h][threadIdx.x];
      cx[threadIdx.x] = (T)t;
    }
    __syncthreads();
  }
  {
    // per axis: even nodes take coarse node x / 2, odd ones the mean of two
    const int X0 = x / 2, X1 = (x & 1) ? (X0 + 1 == nc ? 0 : X0 + 1) : X0;
    const int Y0 = y / 2, Y1 = (y & 1) ? (Y0 + 1 == nc ? 0 : Y0 + 1) : Y0;
    const int Z0 = z / 2, Z1 = (z & 1) ? (Z0 + 1 == nc ? 0 : Z0 + 1) : Z0;
    auto at = [&](int Z, int Y) {
      const int o = (Z * nc + Y) * nc;
      return T(0.5) * (cx[3 * (o + X0) + c] + cx[3 * (o + X1) + c]);
    };
    xx += T(0.5) * (T(0.5) * (at(Z0, Y0) + at(Z0, Y1)) + T(0.5) * (at(Z1, Y0) + at(Z1, Y1)));
  }
  publish(xx);
  r = b - apply();
  d = dv * r * ith;
  xx += d;
  publish(d);
  xx += c1 * d + c2 * dv * (r - apply());
  if (!fine) {
    if (mine) to_global((T *)L.x)[(rhs * 3 + c) * nn + v] = xx;
    return;
  }
  publish(xx);
  // x += P x on the level above: thread (coarse node, component) updates 2^3 nodes
  using T2 = T __attribute__((ext_vector_type(2)));
  const MgLevel &F = mg->lv[l - 1];
  const int nf = F.n;
  if (mine) {
    SHH_GLOBAL T *xf = to_global((T *)F.x) + ((long long)rhs * 3 + c) * F.nn;
    T2 f[2][2];
#pragma unroll
    for (int az = 0; az < 2; ++az)
#pragma unroll
      for (int ay = 0; ay < 2; ++ay)
        f[az][ay] = *(const SHH_GLOBAL T2 *)(xf + ((2 * z + az) * nf + 2 * y + ay) * nf + 2 * x);
    const T *w = vec[c];
#pragma unroll
    for (int az = 0; az < 2; ++az)
#pragma unroll
      for (int ay = 0; ay < 2; ++ay) {
        T e[2];
#pragma unroll
        for (int ix = 0; ix < 2; ++ix) {
          const int X = ix ? xp : x;
          const T a0 = ay ? T(0.5) * (w[(z * n + y) * n + X] + w[(z * n + yp) * n + X]) : w[(z * n + y) * n + X];
          const T a1 = ay ? T(0.5) * (w[(zp * n + y) * n + X] + w[(zp * n + yp) * n + X]) : w[(zp * n + y) * n + X];
          e[ix] = az ? T(0.5) * (a0 + a1) : a0;
        }
        T2 o = f[az][ay];
        o[0] += e[0];
        o[1] += T(0.5) * (e[0] + e[1]);
        *(SHH_GLOBAL T2 *)(xf + ((2 * z + az) * nf + 2 * y + ay) * nf + 2 * x) = o;
      }
  }
}

// The last smoothed level of a design that runs its tail in one launch, or -1
int mg_tail_level(int coarsest, int n_last) { return coarsest >= 2 && n_last == TAIL_N ? coarsest - 1 : -1; }

hipError_t mg_launch_tail(const MgBatch &B, int l, int prec, hipStream_t st) {
  const dim3 g(NRHS, B.count);
  const int fine = l >= 2;  // the voxel level (and the culled solve) restrict into b and read x
  if (prec == 0) mg_tail_kernel<double><<<g, 1024, 0, st>>>(B, l, fine);
  else mg_tail_kernel<float><<<g, 1024, 0, st>>>(B, l, fine);
  return hipGetLastError();
}

}  // namespace shh
