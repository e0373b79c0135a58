// The first coarse level's operator without a stored stencil: q = A_1 v with
// A_1 = P^T K P formed element by element from the eight voxel moduli of each
// coarse element (mixed precision, levels of more than 32^3 nodes).
//
// P restricted to a coarse element is its trilinear interpolation, so the
// coarse element matrix is the integral of the coarse trilinear shape functions
// against the piecewise constant modulus.  With s in [-1, 1] per axis and
//   E(s) = sum_m ehat_m prod_d sgn(s_d)^{m_d}  (ehat: the Hadamard transform of
// the eight moduli, / 8) the 1D integrals in the basis h_s, h_d of hexop.hpp are
// (times 4)
//   value-value:            m = 0: diag(1, 1/3)   m = 1: 1/2 off the diagonal
//   derivative-derivative:  m = 0: (d, d) 4       m = 1: 0
//   derivative-value:       m = 0: (d, s) 2       m = 1: (d, d) 1
// and the element takes 336 multiply-adds for its 24 values.  Checked against
// sum_f E_f Q_f^T K_0 Q_f to rounding.
//
// The tile march is that of stencil.hip on the coarse grid.  Why: the stored
// 27-point stencil is 504 bytes a node, read by each of the four passes of a
// cycle; a pass moved 1 GB for eight 64^3 levels in 200 us, at the memory's
// rate.  The moduli are 32 bytes a node (shared by the load cases) and the
// vectors 36 to 60 per load case; the bound is now the vector ALU (530
// instructions per element and load case).  With it the served batch of eight
// 128^3 designs went from 676 to 591 ms, its setup from 31 to 20 ms (no stencil
// to assemble), one 128^3 design from 60.8 to 55.0 ms; and a level keeps 504
// bytes a node less.  The product is closer to FP64's than that of the stored
// stencil, whose entries are rounded before they cancel: rms error at 96^3, random
// moduli and vectors, nu 0.3, 5.2e-8 -> 3.6e-8 of the largest, nu 0.49 5.6e-7 ->
// 5.2e-7.
#include "kernels.hpp"
#include "mg.hpp"

namespace shh {

namespace {

// y = K_E h without the scale 2 mu / 64 (folded into e): h, y as in hexop.hpp,
// e the moduli's moments, rho = lambda / mu, rho2 = (lambda + 2 mu) / mu
__device__ __forceinline__ void coarse_hex(const float (&e)[8], float rho, float rho2, const float (&h)[3][8],
                                           float (&y)[3][8]) {
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int m = 0; m < 8; ++m) y[c][m] = 0.0f;
  // within a component: the derivatives along axis a
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int b1 = (a + 1) % 3, b2 = (a + 2) % 3;
    const float third = 1.0f / 3.0f;
    const float e0 = 4.0f * e[0], e1 = 2.0f * e[1 << b1], e2 = 2.0f * e[1 << b2], e3 = e[(1 << b1) | (1 << b2)];
    const float e0t = e0 * third, e0n = e0t * third, e1t = e1 * third, e2t = e2 * third;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int p1 = p & 1, p2 = p >> 1, q1 = q & 1, q2 = q >> 1;
        const float w = p1 == q1 ? (p2 == q2 ? (p1 + p2 == 0 ? e0 : (p1 + p2 == 1 ? e0t : e0n)) : (p1 ? e2t : e2))
                                 : (p2 == q2 ? (p2 ? e1t : e1) : e3);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float v = h[c][(1 << a) | (q1 << b1) | (q2 << b2)];
          y[c][(1 << a) | (p1 << b1) | (p2 << b2)] += w * (c == a ? rho2 * v : v);
        }
      }
  }
  // couplings of components i < j, third axis k
  float hl[3][8];  // lambda terms
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int m = 0; m < 8; ++m) hl[c][m] = rho * h[c][m];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const int i = t == 2 ? 1 : 0, j = t == 0 ? 1 : 2, k = 3 - i - j;
#pragma unroll
    for (int ab = 0; ab < 4; ++ab) {
      const int a = ab & 1, b = ab >> 1;
      const float gg = float((2 - a) * (2 - b));
      const float w0 = gg * e[(a << i) | (b << j)], w1 = 0.5f * gg * e[(a << i) | (b << j) | (1 << k)];
      const float w2 = w0 * (1.0f / 3.0f);
      const int A = (a << i) | (1 << j), D = (1 << i) | (b << j);
#pragma unroll
      for (int pq = 0; pq < 4; ++pq) {
        const int p = (pq & 1) << k, q = (pq >> 1) << k;
        const float w = p != q ? w1 : (p ? w2 : w0);
        y[i][D | p] += w * hl[j][A | q];
        y[j][A | p] += w * hl[i][D | q];
        y[i][A | p] += w * h[j][D | q];
        y[j][D | p] += w * h[i][A | q];
      }
    }
  }
}

}  // namespace

template <int TX_, int TY_>
struct CoarseTile {
  static constexpr int X = TX_, Y = TY_, HX = X + 2, HY = Y + 2, EXC = X + 1, EYC = Y + 1;
  static constexpr int NHALO = HX * HY, NELEMC = EXC * EYC, NINT = X * Y, NRING = NHALO - NINT;
  static constexpr int THREADS = 256;
  static_assert(NELEMC <= THREADS && NHALO >= THREADS && NHALO <= 2 * THREADS, "one element, two staged nodes a thread");
};

// grid: 8 XCDs x per; logical workgroup = ((slot * tiles + tile) * nrhs + load
// case); tz: planes a workgroup marches (no sums: the result does not depend on
// the tiling)
template <typename TT, int EP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
void mg_l1_kernel(MgBatch B, int tiles, int per, int nrhs, int tz, int live) {
  constexpr int TX = TT::X, TY = TT::Y, HX = TT::HX, HY = TT::HY, EXC = TT::EXC;
  __shared__ float nbuf[2][3][TT::NHALO];
  __shared__ float ebuf[2][12][TT::NELEMC];
  const int Lg = int(blockIdx.x & 7) * per + int(blockIdx.x >> 3);
  if (Lg >= tiles * nrhs * B.count) return;
  const int rhs = Lg % nrhs, tile = (Lg / nrhs) % tiles, slot = Lg / (nrhs * tiles);
  const SHH_CONST SlotDev *s = to_const(B.slot[slot]);
  const SHH_CONST MgLevel *L = &to_const(B.mg[slot])->lv[1];
  if (live && !to_const(s->st)->active[rhs]) return;
  const int n = L->n, nf = s->n;
  const int tx = (n + TX - 1) / TX, ty = (n + TY - 1) / TY;
  const int tix = tile % tx, tiy = (tile / tx) % ty, tiz = tile / (tx * ty);
  const int x0 = tix * TX, y0 = tiy * TY, z0 = tiz * tz;
  if (z0 >= n) return;
  const int z1 = min(z0 + tz, n);
  const uint32_t plane = (uint32_t)n * (uint32_t)n, cb = plane * (uint32_t)n * 4u;
  const int tid = threadIdx.x;

  const bool is_elem = tid < TT::NELEMC;
  const int ecol = is_elem ? tid : TT::NELEMC - 1;
  const int ecx = ecol % EXC, ecy = ecol / EXC;
  const int ox = tid % TX, oy = tid / TX;
  const bool is_out = tid < TT::NINT && x0 + ox < n && y0 + oy < n;
  const uint32_t ooff = is_out ? ((uint32_t)(y0 + oy) * n + (uint32_t)(x0 + ox)) * 4u : 0u;
  // staging: slot 0 of thread t < NINT its own node, the ring in the others
  const bool ring2 = tid + 256 - TT::NINT < TT::NRING;
  int hslot[2];
  uint32_t hoff[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int j = k == 0 ? tid - TT::NINT : tid + 256 - TT::NINT;
    const int h = k == 0 && tid < TT::NINT ? (oy + 1) * HX + ox + 1 : ring_h<HX, HY>(k == 1 && !ring2 ? 0 : j);
    hslot[k] = h;
    hoff[k] = ((uint32_t)wrapi(y0 - 1 + h / HX, n) * n + (uint32_t)wrapi(x0 - 1 + h % HX, n)) * 4u;
  }
  // the element's 2 x 2 x 2 voxels: four pairs along x
  const uint32_t fplane = (uint32_t)nf * (uint32_t)nf * 4u;
  const uint32_t eoff = (2u * (uint32_t)wrapi(y0 - 1 + ecy, n) * nf + 2u * (uint32_t)wrapi(x0 - 1 + ecx, n)) * 4u;

  const uint64_t vb = 3ull * cb;
  const long long v0 = (long long)rhs * 3 * L->nn;
  auto vec = [&](void *p) { return make_rsrc((const float *)p + v0, vb); };
  const rsrc_t rV = vec(EP == MGE_STEP1 || EP == MGE_LAST ? L->d : (EP == MGE_RES ? L->q : L->x));
  const rsrc_t rE = make_rsrc(s->E32, (uint64_t)fplane * nf), rD = make_rsrc(L->Dinv, vb);
  const rsrc_t rB = vec(L->b), rR = vec(L->r), rX = vec(L->x), rQ = vec(L->q), rDir = vec(L->d);
  const float c1 = (float)L->c1, c2 = (float)L->c2, ith = (float)L->inv_theta;
  const float rho = (float)(s->lam / s->mu), rho2 = (float)((s->lam + 2.0 * s->mu) / s->mu);
  const float scale = (float)(s->mu / 256.0);  // mu, 2 / 64 and the transform's 1 / 8

  using V2 = uint32_t __attribute__((ext_vector_type(2)));
  using F2 = float __attribute__((ext_vector_type(2)));
  float raw[2][3], own[2][3];
  V2 rawE[4];
  auto issue = [&](int z) {
    const uint32_t pz = (uint32_t)wrap1(z, n) * plane * 4u;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (k == 1 && !ring2) continue;
#pragma unroll
      for (int c = 0; c < 3; ++c) raw[k][c] = bload<float>(rV, hoff[k], pz + c * cb);
    }
  };
  auto issueE = [&](int layer) {
    const uint32_t pz = 2u * (uint32_t)wrap1(layer, n) * fplane;
#pragma unroll
    for (int t = 0; t < 4; ++t)
      rawE[t] = __builtin_amdgcn_raw_buffer_load_b64(rE, eoff, pz + (t >> 1) * fplane + (t & 1) * nf * 4u, 0);
  };
  auto finish = [&](int b) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (k == 1 && !ring2) continue;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        nbuf[b][c][hslot[k]] = raw[k][c];
        if (k == 0) own[b][c] = raw[0][c];
      }
    }
  };
  float e[8];
  auto finishE = [&]() {
    float u[8];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const F2 pair = __builtin_bit_cast(F2, rawE[t]);
      const float lo = pair[0], hi = pair[1];
      u[2 * t] = lo + hi;
      u[2 * t + 1] = hi - lo;
    }
#pragma unroll
    for (int d = 1; d < 3; ++d)
#pragma unroll
      for (int m = 0; m < 8; ++m)
        if (!(m & (1 << d))) {
          const float lo = u[m], hi = u[m | (1 << d)];
          u[m] = lo + hi;
          u[m | (1 << d)] = hi - lo;
        }
#pragma unroll
    for (int m = 0; m < 8; ++m) e[m] = scale * u[m];
  };
  auto xy_hadamard = [&](int b, float (&A)[3][4]) {
    const int i00 = ecy * HX + ecx;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float p00 = nbuf[b][c][i00], p10 = nbuf[b][c][i00 + 1];
      const float p01 = nbuf[b][c][i00 + HX], p11 = nbuf[b][c][i00 + HX + 1];
      const float sx0 = p00 + p10, dx0 = p10 - p00, sx1 = p01 + p11, dx1 = p11 - p01;
      A[c][0] = sx0 + sx1;
      A[c][1] = dx0 + dx1;
      A[c][2] = sx1 - sx0;
      A[c][3] = dx1 - dx0;
    }
  };
  float A[3][4], Bc[3][4];
  issue(z0 - 1);
  issueE(z0 - 1);
  finish(0);
  issue(z0);
  __syncthreads();
  xy_hadamard(0, A);
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int m = 0; m < 4; ++m) Bc[c][m] = 0.0f;
  finish(1);
  finishE();
  const int S = z1 - z0 + 1;
  issueE(z0);
  issue(z0 + 1);
  __syncthreads();

  auto step = [&](const int sl, auto bc) {
    constexpr int b = decltype(bc)::value, bn = b ^ 1;
    const int kk = z0 - 1 + sl;
    const uint32_t pk = (uint32_t)kk * plane * 4u;
    // the output node's inputs, loaded while the element work runs
    float op[3], aux[2][3], dv[3];
    if (sl > 0 && is_out) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if constexpr (EP == MGE_STEP1 || EP == MGE_POST) aux[0][c] = bload<float>(rB, ooff, pk + c * cb);
        if constexpr (EP == MGE_RES || EP == MGE_LAST) aux[0][c] = bload<float>(rR, ooff, pk + c * cb);
        if constexpr (EP == MGE_LAST) aux[1][c] = bload<float>(rQ, ooff, pk + c * cb);
        if constexpr (EP != MGE_RES && EP != MGE_NONE) dv[c] = bload<float>(rD, ooff, pk + c * cb);
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) op[c] = own[b][c];
    {
      float An[3][4], h[3][8], y[3][8];
      xy_hadamard(bn, An);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        h[c][0] = 0.0f;  // the rigid mode: never read
#pragma unroll
        for (int m = 1; m < 4; ++m) h[c][m] = A[c][m] + An[c][m];
#pragma unroll
        for (int m = 0; m < 4; ++m) h[c][m + 4] = An[c][m] - A[c][m];
      }
      coarse_hex(e, rho, rho2, h, y);
      float Lo[3][4];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        Lo[c][0] = Bc[c][0] - y[c][4];  // y[c][0] == 0
        Bc[c][0] = y[c][4];
#pragma unroll
        for (int m = 1; m < 4; ++m) {
          Lo[c][m] = Bc[c][m] + (y[c][m] - y[c][m + 4]);
          Bc[c][m] = y[c][m] + y[c][m + 4];
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) A[c][m] = An[c][m];
      }
      if (sl > 0 && is_elem) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float u0 = Lo[c][0] - Lo[c][1], u1 = Lo[c][0] + Lo[c][1], w0 = Lo[c][2] - Lo[c][3],
                      w1 = Lo[c][2] + Lo[c][3];
          ebuf[b][c * 4 + 0][tid] = u0 - w0;
          ebuf[b][c * 4 + 1][tid] = u1 - w1;
          ebuf[b][c * 4 + 2][tid] = u0 + w0;
          ebuf[b][c * 4 + 3][tid] = u1 + w1;
        }
      }
    }
    if (sl + 1 < S) {
      finish(b);
      finishE();
    }
    if (sl + 2 < S) {
      issueE(kk + 2);
      issue(z0 + sl + 2);
    }
    __syncthreads();
    if (sl > 0 && is_out) {
      const int e00 = (oy + 1) * EXC + ox + 1;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float q = (ebuf[b][c * 4 + 0][e00] + ebuf[b][c * 4 + 1][e00 - 1]) +
                        (ebuf[b][c * 4 + 2][e00 - EXC] + ebuf[b][c * 4 + 3][e00 - EXC - 1]);
        const uint32_t o = pk + c * cb;
        // the sweeps of mg_epilogue; op is the operand at the node.  Plain
        // stores: the next pass of the level reads them back soon
        if constexpr (EP == MGE_NONE) {
          bstore<float, 0>(q, rQ, ooff, o);
        } else if constexpr (EP == MGE_STEP1) {
          const float r = aux[0][c] - q, d1 = c1 * op[c] + c2 * dv[c] * r;
          bstore<float, 0>(r, rR, ooff, o);
          bstore<float, 0>(op[c] + d1, rX, ooff, o);
          bstore<float, 0>(d1, rQ, ooff, o);
        } else if constexpr (EP == MGE_RES) {
          bstore<float, 0>(aux[0][c] - q, rR, ooff, o);
        } else if constexpr (EP == MGE_POST) {
          const float r = aux[0][c] - q, d = dv[c] * r * ith;
          bstore<float, 0>(r, rR, ooff, o);
          bstore<float, 0>(d, rDir, ooff, o);
          bstore<float, 0>(op[c] + d, rQ, ooff, o);
        } else {
          bstore<float, 0>(aux[1][c] + c1 * op[c] + c2 * dv[c] * (aux[0][c] - q), rX, ooff, o);
        }
      }
    }
  };
  int sl = 0;
  for (; sl + 1 < S; sl += 2) {
    step(sl, std::integral_constant<int, 0>{});
    step(sl + 1, std::integral_constant<int, 1>{});
  }
  if (sl < S) step(sl, std::integral_constant<int, 0>{});
}

// D^-1 of the level from the moduli: node v is corner a of element v - a, whose
// diagonal there is sum_f E_f G_f[3 a + c][3 a + c]
__global__ __launch_bounds__(256) void mg_l1_diag_kernel(const SlotDev *s, const MgDev *mg) {
  __shared__ float g[8][24];  // diagonals of the child matrices
  const MgLevel &L = mg->lv[1];
  const float *G = (const float *)mg->G;
  for (int t = threadIdx.x; t < 8 * 24; t += 256) g[t / 24][t % 24] = G[(t / 24) * 576 + (t % 24) * 25];
  __syncthreads();
  const unsigned v = blockIdx.x * 256 + threadIdx.x;
  if (v >= (unsigned)L.nn) return;
  const int n = L.n, nf = s->n;
  const unsigned row = v / (unsigned)n;
  const int x = int(v - row * (unsigned)n), y = int(row % (unsigned)n), z = int(row / (unsigned)n);
  double diag[3] = {0.0, 0.0, 0.0};
  for (int a = 0; a < 8; ++a) {
    const int X = wrap1(x - (a & 1), n), Y = wrap1(y - ((a >> 1) & 1), n), Z = wrap1(z - (a >> 2), n);
    for (int f = 0; f < 8; ++f) {
      const long long fe = ((long long)(2 * Z + (f >> 2)) * nf + (2 * Y + ((f >> 1) & 1))) * nf + 2 * X + (f & 1);
      const double e = s->E64[fe];
#pragma unroll
      for (int c = 0; c < 3; ++c) diag[c] += e * (double)g[f][3 * a + c];
    }
  }
  float *Dinv = (float *)L.Dinv;
#pragma unroll
  for (int c = 0; c < 3; ++c) Dinv[c * L.nn + v] = diag[c] > 0.0 ? (float)(1.0 / diag[c]) : 0.0f;
}

hipError_t mg_launch_l1_diag(const SlotDev *d_slot, const MgDev *d_mg, long long nn, hipStream_t st) {
  mg_l1_diag_kernel<<<(unsigned)((nn + 255) / 256), 256, 0, st>>>(d_slot, d_mg);
  return hipGetLastError();
}

namespace {

template <typename TT, int EP>
void launch_l1_tile(const MgBatch &B, int n_max, int nrhs, int live, hipStream_t st) {
  const int txy = ((n_max + TT::X - 1) / TT::X) * ((n_max + TT::Y - 1) / TT::Y);
  // runs that fill whole rounds of the chip's 768 places (three workgroups a
  // CU), a workgroup of tz planes taking tz + 3 layer times
  int tz = 4;
  double best = -1.0;
  for (int t = 4; t <= n_max; ++t) {
    const long long g = (long long)txy * ((n_max + t - 1) / t) * nrhs * B.count;
    const double cost = double((g + 767) / 768) * (t + 3);
    if (best < 0.0 || cost <= best) {
      best = cost;
      tz = t;
    }
  }
  const int tiles = txy * ((n_max + tz - 1) / tz);
  const int per = (tiles * nrhs * B.count + 7) / 8;
  mg_l1_kernel<TT, EP><<<8 * per, 256, 0, st>>>(B, tiles, per, nrhs, tz, live);
}

template <int EP>
void launch_l1(const MgBatch &B, int n_max, int nrhs, int live, hipStream_t st) {
  // 32 x 6 or 24 x 8 nodes, whichever covers the plane in fewer tiles (48^3: 12
  // instead of 16)
  auto count = [n_max](int X, int Y) { return ((n_max + X - 1) / X) * ((n_max + Y - 1) / Y); };
  if (count(32, 6) <= count(24, 8)) launch_l1_tile<CoarseTile<32, 6>, EP>(B, n_max, nrhs, live, st);
  else launch_l1_tile<CoarseTile<24, 8>, EP>(B, n_max, nrhs, live, st);
}

}  // namespace

// n_max: the level's largest n of the batch; nrhs: load cases 0 .. nrhs - 1
hipError_t mg_launch_l1(const MgBatch &B, int n_max, int nrhs, hipStream_t st, int live, int ep) {
  switch (ep) {
    case MGE_STEP1: launch_l1<MGE_STEP1>(B, n_max, nrhs, live, st); break;
    case MGE_RES: launch_l1<MGE_RES>(B, n_max, nrhs, live, st); break;
    case MGE_POST: launch_l1<MGE_POST>(B, n_max, nrhs, live, st); break;
    case MGE_LAST: launch_l1<MGE_LAST>(B, n_max, nrhs, live, st); break;
    default: launch_l1<MGE_NONE>(B, n_max, nrhs, live, st); break;
  }
  return hipGetLastError();
}

}  // namespace shh
