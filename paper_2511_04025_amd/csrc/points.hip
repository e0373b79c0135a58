// The charge field of Eq. (6) at arbitrary points (not voxel centers), and the
// adjoint of a functional of those values: the pieces the fitting objective of
// Eq. (10) needs.  Both go through the trig coefficient tensor of the field
// (see field.hip): F(p) = sum_uvw coef[u][v][w] T_u(x) T_v(y) T_w(z), with
// T_0 = 1, T_{2h-1} = cos 2 pi h s, T_{2h} = sin 2 pi h s.  FP64.
#include "common.hpp"
#include "kernels.hpp"

namespace shh {

// G lanes per point (8 for K <= 3, else 16): the lanes share the point's
// sincospi calls through LDS, then lane u sums its slice of the coefficient
// tensor over v and w, and the lanes add up by shuffles.  (One thread per point
// with its 6 (2K + 1) basis values in scratch memory: 59 us at 4,096 points,
// 64 waves on the chip.)
template <int G>
__global__ __launch_bounds__(256) void points_field_kernel(const SlotDev *s, int npts, const double *pts,
                                                           double *F, double *Gout) {
  constexpr int PP = 256 / G;  // points per workgroup
  constexpr int NBM = G == 8 ? 7 : MAXB;
  __shared__ double coef[NBM * NBM * NBM];
  __shared__ double tv[3][NBM][PP], td[3][NBM][PP];
  const int nb = s->nb, K = s->K;
  const int total = nb * nb * nb;
  for (int e = threadIdx.x; e < total; e += blockDim.x) coef[e] = s->coef[e];
  const int p = threadIdx.x / G, u = threadIdx.x % G;
  const int i = blockIdx.x * PP + p, ic = min(i, npts - 1);
  for (int e = u; e < 3 * (K + 1); e += G) {
    const int ax = e / (K + 1), h = e % (K + 1);
    if (h == 0) {
      tv[ax][0][p] = 1.0;
      td[ax][0][p] = 0.0;
      continue;
    }
    double sn, cs;
    sincospi(2.0 * h * pts[3 * ic + ax], &sn, &cs);
    const double w = 2.0 * M_PI * h;
    tv[ax][2 * h - 1][p] = cs;
    td[ax][2 * h - 1][p] = -w * sn;
    tv[ax][2 * h][p] = sn;
    td[ax][2 * h][p] = w * cs;
  }
  __syncthreads();
  double f = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
  if (u < nb) {
    double t = 0.0, ty = 0.0, tz = 0.0;
    for (int v = 0; v < nb; ++v) {
      double a = 0.0, b = 0.0;
      const double *c = coef + (u * nb + v) * nb;
      for (int w = 0; w < nb; ++w) {
        a += c[w] * tv[2][w][p];
        b += c[w] * td[2][w][p];
      }
      t += tv[1][v][p] * a;
      ty += td[1][v][p] * a;
      tz += tv[1][v][p] * b;
    }
    f = tv[0][u][p] * t;
    gx = td[0][u][p] * t;
    gy = tv[0][u][p] * ty;
    gz = tv[0][u][p] * tz;
  }
#pragma unroll
  for (int off = G / 2; off > 0; off >>= 1) {
    f += __shfl_xor(f, off, 64);
    gx += __shfl_xor(gx, off, 64);
    gy += __shfl_xor(gy, off, 64);
    gz += __shfl_xor(gz, off, 64);
  }
  if (u != 0 || i >= npts) return;
  F[i] = f;
  if (Gout) {
    Gout[i] = gx;
    Gout[npts + i] = gy;
    Gout[2 * npts + i] = gz;
  }
}

// basis values per point: [npts][3][nb]
__global__ __launch_bounds__(256) void points_basis_kernel(int nb, int npts, const double *pts, double *basis) {
  // one thread per point, axis and order h
  const int K1 = (nb + 1) / 2;
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long long)npts * 3 * K1) return;
  const int h = int(e % K1);
  double *b = basis + e / K1 * nb;
  if (h == 0) {
    b[0] = 1.0;
    return;
  }
  double sn, cs;
  sincospi(2.0 * h * pts[e / K1], &sn, &cs);
  b[2 * h - 1] = cs;
  b[2 * h] = sn;
}

// dL/dcoef[u][v][w] = sum_i dL/dF_i T_u(x_i) T_v(y_i) T_w(z_i): one workgroup
// per coefficient, a fixed-order reduction over the points
__global__ __launch_bounds__(256) void points_dcoef_kernel(int nb, int npts, const double *basis, const double *gF,
                                                           double *dcoef) {
  __shared__ double red[16];
  const int e = blockIdx.x;
  const int u = e / (nb * nb), v = (e / nb) % nb, w = e % nb;
  double acc[1] = {0.0};
  for (int i = threadIdx.x; i < npts; i += blockDim.x) {
    const double *b = basis + (long long)i * 3 * nb;
    acc[0] += gF[i] * b[u] * b[nb + v] * b[2 * nb + w];
  }
  block_sum<1>(acc, red, 256);
  if (threadIdx.x == 0) dcoef[e] = acc[0];
}

hipError_t launch_points_field(SlotDev *d_slot, int nb, int npts, const double *d_pts, double *d_F, double *d_G,
                               hipStream_t st) {
  if (nb <= 7) points_field_kernel<8><<<(npts + 31) / 32, 256, 0, st>>>(d_slot, npts, d_pts, d_F, d_G);
  else points_field_kernel<16><<<(npts + 15) / 16, 256, 0, st>>>(d_slot, npts, d_pts, d_F, d_G);
  return hipGetLastError();
}

hipError_t launch_points_dcoef(int nb, int npts, const double *d_pts, const double *d_gF, double *d_basis,
                               double *d_dcoef, hipStream_t st) {
  points_basis_kernel<<<(unsigned)(((long long)npts * 3 * ((nb + 1) / 2) + 255) / 256), 256, 0, st>>>(nb, npts, d_pts,
                                                                                                 d_basis);
  points_dcoef_kernel<<<nb * nb * nb, 256, 0, st>>>(nb, npts, d_basis, d_gF, d_dcoef);
  return hipGetLastError();
}

}  // namespace shh
