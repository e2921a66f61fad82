// Setup and per-potential operator kernels.
//
//  reference element   GLL/Gauss rules and 1-D Lagrange tables (host, a few
//                      numbers), 3-D basis/gradient tables, cell stiffness and
//                      lumped GLL mass on the GPU (Sec. III.A)
//  enrichment          normalization, b = int N phi, kinetic part of
//                      B = <phi| -1/2 Lap |N>, M^phiphi, kinetic H^phiphi,
//                      C = b diag(m)^-1, M^ee = M^phiphi - b diag(m)^-1 b^T and
//                      the inverses of its atom blocks (Sec. II.B, Eq.
//                      MEInvApprox)
//  projectors          P^C = int beta N, P^phi = int beta phi, D (Eq. KS)
//  potential           cell Hamiltonians 1/2 K + N^T diag(w v) N in the MFMA
//                      operand layout, B and H^phiphi potential parts
#include <cmath>
#include <limits>
#include <vector>

#include "efe_device.h"
#include "line_ops.h"

// ------------------------------------------------------------ 1-D rules
// T = double, and long double for tables that are rounded once (cell_tp.hip)
template <class T>
static void legendre(int n, T x, T &P, T &dP) {
  T p0 = 1.0, p1 = x;
  if (n == 0) {
    P = 1.0;
    dP = 0.0;
    return;
  }
  for (int k = 1; k < n; ++k) {
    T p2 = ((2 * k + 1) * x * p1 - k * p0) / (k + 1);
    p0 = p1;
    p1 = p2;
  }
  P = p1;
  dP = n * (x * p1 - p0) / (x * x - T(1.0));
}

template <class T>
static void gll_rule(int p, std::vector<T> &x, std::vector<T> &w) {
  x.assign(p + 1, 0.0);
  w.assign(p + 1, 0.0);
  x[0] = -1.0;
  x[p] = 1.0;
  for (int i = 1; i < p; ++i) {
    T t = -cos(M_PI * i / p);
    for (int it = 0; it < 100; ++it) {   // Newton on P_p'
      T P, dP;
      legendre(p, t, P, dP);
      T d2P = (2 * t * dP - p * (p + 1) * P) / (T(1.0) - t * t);
      T dt = dP / d2P;
      t -= dt;
      if (std::abs(dt) < std::min<T>(1e-16, std::numeric_limits<T>::epsilon())) break;
    }
    x[i] = t;
  }
  for (int i = 0; i <= p; ++i) {
    T P, dP;
    legendre(p, x[i], P, dP);
    w[i] = T(2.0) / (p * (p + 1) * P * P);
  }
}

template <class T>
static void gauss_rule(int n, std::vector<T> &x, std::vector<T> &w) {
  x.assign(n, 0.0);
  w.assign(n, 0.0);
  for (int i = 0; i < n; ++i) {
    T t = -cos(M_PI * (i + 0.75) / (n + 0.5));
    for (int it = 0; it < 100; ++it) {
      T P, dP;
      legendre(n, t, P, dP);
      T dt = P / dP;
      t -= dt;
      if (std::abs(dt) < std::min<T>(1e-16, std::numeric_limits<T>::epsilon())) break;
    }
    T P, dP;
    legendre(n, t, P, dP);
    x[i] = t;
    w[i] = T(2.0) / ((T(1.0) - t * t) * dP * dP);
  }
}

// values and derivatives of the Lagrange basis on xg at the points xq
template <class T>
static void lagrange(const std::vector<T> &xg, const std::vector<T> &xq, std::vector<T> &N1,
                     std::vector<T> &D1) {
  const int P = (int)xg.size(), nq = (int)xq.size();
  N1.resize(nq * P);
  D1.resize(nq * P);
  for (int q = 0; q < nq; ++q)
    for (int a = 0; a < P; ++a) {
      T v = 1.0, d = 0.0;
      for (int b = 0; b < P; ++b)
        if (b != a) v *= (xq[q] - xg[b]) / (xg[a] - xg[b]);
      for (int b = 0; b < P; ++b) {
        if (b == a) continue;
        T t = T(1.0) / (xg[a] - xg[b]);
        for (int cc = 0; cc < P; ++cc)
          if (cc != a && cc != b) t *= (xq[q] - xg[cc]) / (xg[a] - xg[cc]);
        d += t;
      }
      N1[q * P + a] = v;
      D1[q * P + a] = d;
    }
}

// ------------------------------------------------------------ kernels
// 3-D basis values and physical gradients at the Gauss points, weights.
__global__ void k_ref3d(int P, int nq, const double *__restrict__ N1, const double *__restrict__ D1,
                        const double *__restrict__ wq, double hx, double hy, double hz,
                        double *__restrict__ N3, double *__restrict__ G3, double *__restrict__ W3) {
  const int nloc = P * P * P, nqp = nq * nq * nq;
  int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= (int64_t)nqp * nloc) return;
  int q = idx / nloc, l = idx % nloc;
  int a = l % P, b = (l / P) % P, c = l / (P * P);
  int qa = q % nq, qb = (q / nq) % nq, qc = q / (nq * nq);
  double na = N1[qa * P + a], nb = N1[qb * P + b], nc = N1[qc * P + c];
  double da = D1[qa * P + a], db = D1[qb * P + b], dc = D1[qc * P + c];
  N3[idx] = na * nb * nc;
  G3[idx] = da * nb * nc * (2.0 / hx);
  G3[(int64_t)nqp * nloc + idx] = na * db * nc * (2.0 / hy);
  G3[2 * (int64_t)nqp * nloc + idx] = na * nb * dc * (2.0 / hz);
  if (l == 0) W3[q] = wq[qa] * wq[qb] * wq[qc] * (hx * hy * hz / 8.0);
}

// K[l][l'] = sum_q W_q grad N_l . grad N_l'
__global__ void k_stiffness(int nloc, int nqp, const double *__restrict__ G3,
                            const double *__restrict__ W3, double *__restrict__ K) {
  int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= (int64_t)nloc * nloc) return;
  int i = idx / nloc, j = idx % nloc;
  const int64_t s = (int64_t)nqp * nloc;
  double acc = 0.0;
  for (int q = 0; q < nqp; ++q) {
    const int64_t o = (int64_t)q * nloc;
    acc += W3[q] * (G3[o + i] * G3[o + j] + G3[s + o + i] * G3[s + o + j] +
                    G3[2 * s + o + i] * G3[2 * s + o + j]);
  }
  K[idx] = acc;
}

// Lumped GLL mass: product of 1-D lumped weights (shared nodes get both cells).
__global__ void k_lumped_mass(int64_t n1x, int64_t n1y, int64_t n1z, int p,
                              const double *__restrict__ wg, double hx, double hy, double hz,
                              double *__restrict__ m, double *__restrict__ minv,
                              double *__restrict__ m_int) {
  int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (n >= n1x * n1y * n1z) return;
  int64_t idx[3] = {n % n1x, (n / n1x) % n1y, n / (n1x * n1y)};
  int64_t nn[3] = {n1x, n1y, n1z};
  double hh[3] = {hx, hy, hz};
  double mm = 1.0;
  bool bnd = false;
  for (int d = 0; d < 3; ++d) {
    int64_t i = idx[d];
    int a = (int)(i % p);
    double w;
    if (a == 0 && i > 0 && i < nn[d] - 1) w = wg[0] + wg[p];
    else if (i == nn[d] - 1) w = wg[p];
    else w = wg[a];
    mm *= 0.5 * hh[d] * w;
    if (i == 0 || i == nn[d] - 1) bnd = true;
  }
  m[n] = mm;
  minv[n] = bnd ? 0.0 : 1.0 / mm;
  m_int[n] = bnd ? 0.0 : mm;
}

// sum_q W phi_raw^2 per enrichment function (one block per (atom, cell) pair)
__global__ void k_enr_norm(MeshGeo g, EnrParam e, const double *__restrict__ xq1,
                           const double *__restrict__ W3, const double *__restrict__ xyz,
                           const int32_t *__restrict__ pair_atom,
                           const int32_t *__restrict__ pair_cell, double *__restrict__ norm2) {
  __shared__ double red[256][9];
  const int pr = blockIdx.x;
  const int I = pair_atom[pr], cell = pair_cell[pr];
  double acc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int q = threadIdx.x; q < g.nqp; q += blockDim.x) {
    double x[3], phi[9];
    quad_point(g, xq1, cell, q, x);
    enr_eval(e, x[0] - xyz[3 * I], x[1] - xyz[3 * I + 1], x[2] - xyz[3 * I + 2], phi, nullptr);
    for (int k = 0; k < e.nf; ++k) acc[k] += W3[q] * phi[k] * phi[k];
  }
  for (int k = 0; k < 9; ++k) red[threadIdx.x][k] = acc[k];
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s)
      for (int k = 0; k < 9; ++k) red[threadIdx.x][k] += red[threadIdx.x + s][k];
    __syncthreads();
  }
  if (threadIdx.x < (unsigned)e.nf) atomicAdd(&norm2[I * e.nf + threadIdx.x], red[0][threadIdx.x]);
}

__global__ void k_inv_sqrt(int64_t n, double *__restrict__ x) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) x[i] = 1.0 / sqrt(x[i]);
}

// Per pair: b[l][k] += sum_q W phi_k N_l ; Bkin[l][k] += 1/2 sum_q W grad phi_k . grad N_l
// (with_kin) or, for the potential part, Bv[l][k] += sum_q W v phi_k N_l.
template <bool KIN>
__global__ __launch_bounds__(256) void k_enr_pair_proj(
    MeshGeo g, EnrParam e, const double *__restrict__ xq1, const double *__restrict__ W3,
    const double *__restrict__ N3, const double *__restrict__ G3, const double *__restrict__ xyz,
    const double *__restrict__ nu, const int32_t *__restrict__ pair_atom,
    const int32_t *__restrict__ pair_cell, const int32_t *__restrict__ lmap,
    const double *__restrict__ vq, double *__restrict__ out_b, double *__restrict__ out_k,
    double *__restrict__ out_pair) {
  // weighted values at up to 64 quadrature points at a time
  __shared__ double sphi[9][64];
  __shared__ double sgrad[3][9][64];
  const int pr = blockIdx.x;
  const int I = pair_atom[pr], cell = pair_cell[pr];
  const int nf = e.nf, nloc = g.nloc, nqp = g.nqp;
  const int64_t s3 = (int64_t)nqp * nloc;
  // each thread owns outputs (l, k) with l = tid + 256 * r
  double accb[2][9], acck[2][9];
  for (int r = 0; r < 2; ++r)
    for (int k = 0; k < 9; ++k) accb[r][k] = acck[r][k] = 0.0;
  for (int q0 = 0; q0 < nqp; q0 += 64) {
    const int nqc = min(64, nqp - q0);
    if (threadIdx.x < (unsigned)nqc) {
      const int q = q0 + threadIdx.x;
      double x[3], phi[9], grad[27];
      quad_point(g, xq1, cell, q, x);
      enr_eval(e, x[0] - xyz[3 * I], x[1] - xyz[3 * I + 1], x[2] - xyz[3 * I + 2], phi,
               KIN ? grad : nullptr);
      const double w = W3[q] * (KIN ? 1.0 : vq[(int64_t)cell * nqp + q]);
      for (int k = 0; k < nf; ++k) {
        const double s = nu[I * nf + k];
        sphi[k][threadIdx.x] = w * s * phi[k];
        if (KIN)
          for (int d = 0; d < 3; ++d) sgrad[d][k][threadIdx.x] = 0.5 * w * s * grad[3 * k + d];
      }
    }
    __syncthreads();
    for (int r = 0; r < 2; ++r) {
      const int l = threadIdx.x + 256 * r;
      if (l >= nloc) continue;
      for (int qq = 0; qq < nqc; ++qq) {
        const int64_t o = (int64_t)(q0 + qq) * nloc + l;
        const double n = N3[o];
        for (int k = 0; k < nf; ++k) accb[r][k] += sphi[k][qq] * n;
        if (KIN) {
          const double gx = G3[o], gy = G3[s3 + o], gz = G3[2 * s3 + o];
          for (int k = 0; k < nf; ++k)
            acck[r][k] += sgrad[0][k][qq] * gx + sgrad[1][k][qq] * gy + sgrad[2][k][qq] * gz;
        }
      }
    }
    __syncthreads();
  }
  for (int r = 0; r < 2; ++r) {
    const int l = threadIdx.x + 256 * r;
    if (l >= nloc) continue;
    // the cell's own block (kinetic part), kept per pair for the coupling
    // E_c = B_c - C_c H_c of the orthogonalized basis
    if (KIN && out_pair)
      for (int k = 0; k < nf; ++k) out_pair[((int64_t)pr * nloc + l) * nf + k] = acck[r][k];
    const int32_t s = lmap[(int64_t)pr * nloc + l];
    if (s < 0) continue;
    for (int k = 0; k < nf; ++k) {
      atomicAdd(&out_b[(int64_t)s * nf + k], accb[r][k]);
      if (KIN) atomicAdd(&out_k[(int64_t)s * nf + k], acck[r][k]);
    }
  }
}

// Potential part of the same projections, on FP64 MFMA: for one (atom, cell)
// pair, out[l][k] += sum_q N[q][l] (w v s_k phi_k)(x_q), a 343 x 9 product
// over the cell's Gauss points.  The weighted enrichment values sit in LDS as
// the B operand (16 columns, zero past nf and past nqp); each wave takes row
// blocks of N^T (A operand, 16 consecutive entries of a row of N per load).
typedef double v4d_p __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void k_enr_pair_proj_v(
    MeshGeo g, EnrParam e, const double *__restrict__ xq1, const double *__restrict__ W3,
    const double *__restrict__ N3, const double *__restrict__ xyz, const double *__restrict__ nu,
    const int32_t *__restrict__ pair_atom, const int32_t *__restrict__ pair_cell,
    const int32_t *__restrict__ lmap, const double *__restrict__ vq, int KQ,
    double *__restrict__ out_b, const double *__restrict__ kin_pair,
    double *__restrict__ out_pair) {
  extern __shared__ double sphi[];   // [4 KQ][16]
  const int pr = blockIdx.x;
  const int I = pair_atom[pr], cell = pair_cell[pr];
  const int nf = e.nf, nloc = g.nloc, nqp = g.nqp;
  for (int q = threadIdx.x; q < 4 * KQ; q += blockDim.x) {
    double row[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) row[k] = 0.0;
    if (q < nqp) {
      double x[3], phi[9];
      quad_point(g, xq1, cell, q, x);
      enr_eval(e, x[0] - xyz[3 * I], x[1] - xyz[3 * I + 1], x[2] - xyz[3 * I + 2], phi, nullptr);
      const double w = W3[q] * vq[(int64_t)cell * nqp + q];
#pragma unroll
      for (int k = 0; k < 9; ++k)
        if (k < nf) row[k] = w * nu[I * nf + k] * phi[k];
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) sphi[q * 16 + k] = row[k];
  }
  __syncthreads();
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, li = lane % 16, lk = lane / 16;
  const int RB = (nloc + 15) / 16;
  for (int rb = wave; rb < RB; rb += 4) {
    const double *np = N3 + min(16 * rb + li, nloc - 1);
    v4d_p acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int ks = 0; ks < KQ; ++ks) {
      const int q = min(4 * ks + lk, nqp - 1);   // past nqp: zero rows of sphi
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(np[(int64_t)q * nloc],
                                                 sphi[(4 * ks + lk) * 16 + li], acc, 0, 0, 0);
    }
    // accumulator v of lane l: local node 16 rb + 4 v + l/16, function l%16
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int l = 16 * rb + 4 * v + lk;
      if (l < nloc && li < nf) {
        const int64_t o = ((int64_t)pr * nloc + l) * nf + li;
        if (out_pair) out_pair[o] = kin_pair[o] + acc[v];
        const int32_t sn = lmap[(int64_t)pr * nloc + l];
        if (sn >= 0) atomicAdd(&out_b[(int64_t)sn * nf + li], acc[v]);
      }
    }
  }
}

// The same by 1-D contractions where the Gauss rule allows them (nq = P): the
// weighted enrichment values sit in LDS, function by function, and each axis
// goes back to the nodes by N~^T = (diag(sqrt(w h/2)) N)^T along its lines, so the
// values carry sqrt(W) here.  9 x 3 x P^4 multiply-adds a pair instead of 16 P^6
// on the matrix cores; evaluating the functions and the atomics are what is left
// (64 atoms: 0.43 ms, 4.6 before).
constexpr int PAIR_TP_T = 192;
template <int P>
__global__ __launch_bounds__(PAIR_TP_T) void k_enr_pair_proj_tp(
    MeshGeo g, EnrParam e, const double *__restrict__ xq1, const double *__restrict__ W3,
    const double *tpm, const double *__restrict__ xyz, const double *__restrict__ nu,
    const int32_t *__restrict__ pair_atom, const int32_t *__restrict__ pair_cell,
    const int32_t *__restrict__ lmap, const double *__restrict__ vq, double *__restrict__ out_b,
    const double *__restrict__ kin_pair, double *__restrict__ out_pair) {
  constexpr int PP = P * P, N = P * P * P;
  __shared__ double L[9][N];
  const int pr = blockIdx.x, t = threadIdx.x;
  const int I = pair_atom[pr], cell = pair_cell[pr];
  const int nf = e.nf;
  for (int q = t; q < N; q += PAIR_TP_T) {
    double x[3], phi[9];
    quad_point(g, xq1, cell, q, x);
    enr_eval(e, x[0] - xyz[3 * I], x[1] - xyz[3 * I + 1], x[2] - xyz[3 * I + 2], phi, nullptr);
    const double w = sqrt(W3[q]) * vq[(int64_t)cell * N + q];
#pragma unroll
    for (int k = 0; k < 9; ++k)
      if (k < nf) L[k][q] = w * nu[I * nf + k] * phi[k];
  }
  cdouble *const m0 = (cdouble *)(uintptr_t)tpm;
#pragma unroll
  for (int d = 2; d >= 0; --d) {
    const int st = d == 0 ? 1 : d == 1 ? P : PP;
    cdouble *m = fresh(m0);
    __syncthreads();
    for (int i = t; i < nf * PP; i += PAIR_TP_T) {
      const int k = i / PP, j = i % PP;
      double *p = &L[k][d == 0 ? j * P : d == 1 ? j / P * PP + j % P : j];
      double v[P], y[P];
#pragma unroll
      for (int n = 0; n < P; ++n) v[n] = p[n * st];
      mul1d<P, true>(m, d, v, y);
#pragma unroll
      for (int n = 0; n < P; ++n) p[n * st] = y[n];
    }
  }
  __syncthreads();
  for (int i = t; i < N * nf; i += PAIR_TP_T) {
    const int l = i / nf, k = i % nf;
    const double b = L[k][l];
    const int64_t o = (int64_t)pr * N * nf + i;
    if (out_pair) out_pair[o] = kin_pair[o] + b;
    const int32_t sn = lmap[(int64_t)pr * N + l];
    if (sn >= 0) atomicAdd(&out_b[(int64_t)sn * nf + k], b);
  }
}

// C = b / m on support nodes
__global__ void k_scale_by_minv(int64_t n_snodes, int nf, const int32_t *__restrict__ snode,
                                const double *__restrict__ minv, const double *__restrict__ b,
                                double *__restrict__ C) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n_snodes * nf) return;
  C[i] = b[i] * minv[snode[i / nf]];
}

// group-major copy: dst[(slot nf + k) 8 + n % 8] = src[nm_src[e] nf + k] for
// every node-major entry e of node n (slot = its atom's place in the union of
// the atoms of the 8-node group of n); entries not written stay zero
__global__ void k_to_group_major(int64_t n_nodes, int nf, const int32_t *__restrict__ nm_ptr,
                                 const int32_t *__restrict__ nm_src,
                                 const int32_t *__restrict__ nm_gslot,
                                 const double *__restrict__ src, double *__restrict__ dst) {
  const int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (n >= n_nodes) return;
  const int j = (int)(n & 7);
  for (int32_t e = nm_ptr[n]; e < nm_ptr[n + 1]; ++e) {
    const int64_t slot = nm_gslot[e], s0 = (int64_t)nm_src[e] * nf;
    for (int k = 0; k < nf; ++k) dst[(slot * nf + k) * 8 + j] = src[s0 + k];
  }
}

// Per (cell, I, J): M[I k][J l] += sum_q W phi_Ik phi_Jl and
// H[I k][J l] += 1/2 sum_q W grad phi_Ik . grad phi_Jl.
__global__ __launch_bounds__(128) void k_enr_pp(MeshGeo g, EnrParam e, const double *__restrict__ xq1,
                                                const double *__restrict__ W3,
                                                const double *__restrict__ xyz,
                                                const double *__restrict__ nu,
                                                const int32_t *__restrict__ trip,
                                                int64_t n_enr,
                                                double *__restrict__ M, double *__restrict__ H) {
  __shared__ double pI[4][9][64], pJ[4][9][64];
  const int64_t t = blockIdx.x;
  const int cell = trip[3 * t], I = trip[3 * t + 1], J = trip[3 * t + 2];
  const int nf = e.nf, nqp = g.nqp;
  const int tid = threadIdx.x;
  const int k = tid / 9, l = tid % 9;          // 81 output pairs
  double am = 0.0, ah = 0.0;
  for (int q0 = 0; q0 < nqp; q0 += 64) {
    const int nqc = min(64, nqp - q0);
    if (tid < nqc) {
      const int q = q0 + tid;
      double x[3], phi[9], grad[27], phj[9], grj[27];
      quad_point(g, xq1, cell, q, x);
      enr_eval(e, x[0] - xyz[3 * I], x[1] - xyz[3 * I + 1], x[2] - xyz[3 * I + 2], phi,
               grad);
      enr_eval(e, x[0] - xyz[3 * J], x[1] - xyz[3 * J + 1], x[2] - xyz[3 * J + 2], phj,
               grj);
      const double w = W3[q];
      for (int a = 0; a < nf; ++a) {
        const double si = nu[I * nf + a], sj = nu[J * nf + a];
        pI[0][a][tid] = w * si * phi[a];
        pJ[0][a][tid] = sj * phj[a];
        for (int d = 0; d < 3; ++d) {
          pI[1 + d][a][tid] = 0.5 * w * si * grad[3 * a + d];
          pJ[1 + d][a][tid] = sj * grj[3 * a + d];
        }
      }
    }
    __syncthreads();
    if (k < nf && l < nf) {
      for (int qq = 0; qq < nqc; ++qq) {
        am += pI[0][k][qq] * pJ[0][l][qq];
        ah += pI[1][k][qq] * pJ[1][l][qq] + pI[2][k][qq] * pJ[2][l][qq] +
              pI[3][k][qq] * pJ[3][l][qq];
      }
    }
    __syncthreads();
  }
  if (k < nf && l < nf) {
    const int64_t o = (int64_t)(I * nf + k) * n_enr + J * nf + l;
    atomicAdd(&M[o], am);
    atomicAdd(&H[o], ah);
  }
}

// Potential part of H^phiphi, H[I k][J l] += sum_q W v phi_Ik phi_Jl over one
// cell and two blocks of its atoms (up to 96 functions each), on FP64 MFMA: the
// functions are evaluated once a cell, not once a pair of atoms, and sit in LDS
// for 32 Gauss points at a time; the four waves share the 16 x 16 products out.
// A block with itself takes the upper triangle of products and mirrors it (64
// atoms: 0.53 ms; a work-group per pair of atoms with scalar products 3.9).
constexpr int PPV_F = EFE_PPV_F, PPV_Q = 32, PPV_LD = PPV_Q + 4;
constexpr int PPV_T = PPV_F / 16 * (PPV_F / 16) / 4;   // products of a wave
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_enr_ppv(MeshGeo g, EnrParam e, const double *__restrict__ xq1, const double *__restrict__ W3,
               const double *__restrict__ xyz, const double *__restrict__ nu,
               const int32_t *__restrict__ items, const int32_t *__restrict__ trip,
               const double *__restrict__ vq, int64_t n_enr, double *__restrict__ H) {
  __shared__ double S[2][PPV_F * PPV_LD];
  __shared__ double ws[PPV_Q];
  const int32_t *it = items + 4 * (int64_t)blockIdx.x;
  const int t0 = it[0], n = it[1], nf = e.nf, nqp = g.nqp;
  const int ab = PPV_F / nf, a0 = it[2] * ab, b0 = it[3] * ab;   // first atoms of the blocks
  const bool diag = a0 == b0;
  const int na = min(ab, n - a0), nb = min(ab, n - b0);
  const int cell = trip[3 * (int64_t)t0];
  auto atom = [&](int i) { return trip[3 * ((int64_t)t0 + i) + 2]; };
  const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t / 64), lane = t % 64;
  const int li = lane % 16, lk = lane / 16;
  const int Fa = na * nf, Fb = nb * nf, Ra = (Fa + 15) / 16, Rb = (Fb + 15) / 16;
  // this wave's products: every fourth of the list of (row block, column block)
  int rr[PPV_T], cc[PPV_T], m = 0;
  v4d_p acc[PPV_T];
  {
    int id = 0;
#pragma unroll
    for (int i = 0; i < PPV_T; ++i) {
      rr[i] = cc[i] = -1;
      acc[i] = (v4d_p){0.0, 0.0, 0.0, 0.0};
    }
    for (int r = 0; r < Ra; ++r)
      for (int c = diag ? r : 0; c < Rb; ++c, ++id)
        if (id % 4 == wave) {
#pragma unroll
          for (int i = 0; i < PPV_T; ++i)
            if (i == m) {
              rr[i] = r;
              cc[i] = c;
            }
          ++m;
        }
  }
  // rows past the functions stay zero
  for (int i = t; i < 2 * PPV_F * PPV_LD; i += 256) (&S[0][0])[i] = 0.0;
  const double *const SB = diag ? S[0] : S[1];
  const int nall = diag ? na : na + nb;
  for (int q0 = 0; q0 < nqp; q0 += PPV_Q) {
    __syncthreads();
    if (t < PPV_Q) ws[t] = q0 + t < nqp ? W3[q0 + t] * vq[(int64_t)cell * nqp + q0 + t] : 0.0;
    for (int i = t; i < nall * PPV_Q; i += 256) {
      const int q = i % PPV_Q, a = i / PPV_Q, I = atom(a < na ? a0 + a : b0 + a - na);
      double x[3], phi[9];
      quad_point(g, xq1, cell, min(q0 + q, nqp - 1), x);   // past nqp: weight 0
      enr_eval(e, x[0] - xyz[3 * I], x[1] - xyz[3 * I + 1], x[2] - xyz[3 * I + 2], phi, nullptr);
      double *dst = (a < na ? S[0] + a * nf * PPV_LD : S[1] + (a - na) * nf * PPV_LD) + q;
#pragma unroll
      for (int k = 0; k < 9; ++k)
        if (k < nf) dst[k * PPV_LD] = nu[I * nf + k] * phi[k];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PPV_T; ++i)
      if (i < m) {
        const double *pa = S[0] + (16 * rr[i] + li) * PPV_LD + lk;
        const double *pb = SB + (16 * cc[i] + li) * PPV_LD + lk;
#pragma unroll
        for (int s = 0; s < PPV_Q / 4; ++s)
          acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[4 * s] * ws[4 * s + lk], pb[4 * s],
                                                        acc[i], 0, 0, 0);
      }
  }
#pragma unroll
  for (int i = 0; i < PPV_T; ++i)
    if (i < m)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int f = 16 * rr[i] + 4 * v + lk, h = 16 * cc[i] + li;
        if (f >= Fa || h >= Fb) continue;
        const int64_t r = (int64_t)atom(a0 + f / nf) * nf + f % nf;
        const int64_t c = (int64_t)atom(b0 + h / nf) * nf + h % nf;
        atomicAdd(&H[r * n_enr + c], acc[i][v]);
        if (!diag || rr[i] != cc[i]) atomicAdd(&H[c * n_enr + r], acc[i][v]);
      }
}

// Row f of b diag(m)^-1 b^T, subtracted from M^phiphi: Mee[f][:] = Mpp[f][:] - acc
__global__ __launch_bounds__(256) void k_mee_rows(int nf, int64_t n_enr, const int32_t *__restrict__ snode_ptr,
                                                  const int32_t *__restrict__ snode,
                                                  const int32_t *__restrict__ nm_ptr,
                                                  const int32_t *__restrict__ nm_atom,
                                                  const int32_t *__restrict__ nm_src,
                                                  const double *__restrict__ C_am,
                                                  const double *__restrict__ b_am,
                                                  const double *__restrict__ Mpp,
                                                  double *__restrict__ Mee) {
  extern __shared__ double acc[];
  const int64_t f = blockIdx.x;
  const int I = f / nf, k = f % nf;
  for (int64_t i = threadIdx.x; i < n_enr; i += blockDim.x) acc[i] = 0.0;
  __syncthreads();
  for (int32_t s = snode_ptr[I] + threadIdx.x; s < snode_ptr[I + 1]; s += blockDim.x) {
    const int32_t j = snode[s];
    const double cf = C_am[(int64_t)s * nf + k];
    for (int32_t ee = nm_ptr[j]; ee < nm_ptr[j + 1]; ++ee) {
      const int J = nm_atom[ee];
      const int64_t src = nm_src[ee];
      for (int l = 0; l < nf; ++l) atomicAdd(&acc[J * nf + l], cf * b_am[src * nf + l]);
    }
  }
  __syncthreads();
  for (int64_t i = threadIdx.x; i < n_enr; i += blockDim.x)
    Mee[f * n_enr + i] = Mpp[f * n_enr + i] - acc[i];
}

// Coupling of the orthogonalized basis, E_c = B_c - C_c H_c of every (atom, cell)
// pair (Sec. II.B: N^E = phi - C N^C), in FP64 from the dense cell Hamiltonians.
// 1-D contractions do it in 1.3 ms for 64 atoms, but B - C H cancels most of its
// digits, what is left enters G and with it every step of a filter, and the
// output of degree 40 moved by 6e-9.  One work-group takes a cell and 32 of its
// enrichment functions: C_c^T (nodes x 32) in LDS, each wave every eighth 16 rows
// of H_c, whose fragments feed two products (one for the last 16 functions or
// fewer).  Bound by the reading of H_c, with one work-group a CU to cover it: eight
// fragments are on their way while eight are multiplied, and the work-groups of a
// cell run on one XCD, whose L2 they share (64 atoms: 3.0 ms, 7.8 with the loads
// before their products and a cell spread over the XCDs; 27 atoms of 4 functions at
// p = 6: 0.55 ms, 1.23, and 0.93 as 16 functions a work-group).
//
// EC (no cell couples to more than 32 functions): the work-group holds E_c and C_c
// of the whole cell, and H^E_ee -= E_c C_c^T is formed on the way, four products more
// per 16 nodes whose operand is the accumulator as it stands (two atoms on 5^3
// cells: the 12.5 us of k_hee_box less).
template <bool EC>
__global__ __launch_bounds__(512) void k_build_E(
    int64_t ncells, int nloc, int RB, int KS, int nf, int max_cb, const double *__restrict__ Ht,
    const int32_t *__restrict__ eptr, const int32_t *__restrict__ epair,
    const int32_t *__restrict__ lmap, const int32_t *__restrict__ spair,
    const double *__restrict__ C_am, const double *__restrict__ B_pair, double *__restrict__ E,
    const int32_t *__restrict__ atom, int64_t n_enr, double *__restrict__ Hee) {
  __shared__ double Cs[2][EFE_MAXLOC + 16][16];
  __shared__ double Hs[EC ? 32 : 1][33];
  const int slot = blockIdx.x / 8, cb = slot % max_cb;
  const int64_t cell = (int64_t)(slot / max_cb) * 8 + blockIdx.x % 8;
  if (cell >= ncells) return;
  const int32_t p0 = eptr[cell];
  const int ne = (eptr[cell + 1] - p0) * nf;
  if (32 * cb >= ne) return;
  const bool two = ne - 32 * cb > 16;
  if constexpr (EC)
    for (int i = threadIdx.x; i < 32 * 33; i += 512) Hs[i / 33][i % 33] = 0.0;
  for (int i = threadIdx.x; i < (EC ? 16 * RB : 4 * KS) * 32; i += 512) {
    const int l = i / 32, j = i % 32, e = 32 * cb + j;
    double v = 0.0;
    if (l < nloc && e < ne) {
      const int32_t sn = lmap[(int64_t)epair[p0 + e / nf] * nloc + l];
      if (sn >= 0) v = C_am[(int64_t)sn * nf + e % nf];
    }
    Cs[j / 16][l][j % 16] = v;
  }
  __syncthreads();
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, li = lane % 16, lk = lane / 16;
  v4d_p hc[2][2];
  if constexpr (EC)
#pragma unroll
    for (int b = 0; b < 4; ++b) hc[b / 2][b % 2] = (v4d_p){0.0, 0.0, 0.0, 0.0};
  for (int rb = wave; rb < RB; rb += 8) {
    const double *hp = Ht + (cell * RB + rb) * KS * 64 + lane;
    v4d_p acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
    constexpr int U = 8;
    double h0[U], h1[U];
    auto load = [&](int k0, double (&h)[U]) {
#pragma unroll
      for (int u = 0; u < U; ++u) h[u] = hp[(int64_t)min(k0 + u, KS - 1) * 64];
    };
    auto multiply = [&](int k0, const double (&h)[U]) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int ks = k0 + u;
        if (ks >= KS) break;
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(h[u], Cs[0][4 * ks + lk][li], acc[0], 0, 0, 0);
        if (two)
          acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(h[u], Cs[1][4 * ks + lk][li], acc[1], 0, 0, 0);
      }
    };
    load(0, h0);
    for (int k0 = 0; k0 < KS; k0 += 2 * U) {
      load(k0 + U, h1);
      multiply(k0, h0);
      load(k0 + 2 * U, h0);
      multiply(k0 + U, h1);
    }
    // accumulator v of lane l: node row 16 rb + 4 v + l/16, function l%16
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int e = 32 * cb + 16 * b + li;
      if (e >= ne) continue;   // acc is zero there: so is C
      const int64_t pr = epair[p0 + e / nf];
      const int32_t sp = spair[pr];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int l = 16 * rb + 4 * v + lk;
        if (l >= nloc) continue;
        // B_c vanishes on the layer of cells outside the support
        const double bv = sp >= 0 ? B_pair[((int64_t)sp * nloc + l) * nf + e % nf] : 0.0;
        acc[b][v] = bv - acc[b][v];
        E[(pr * nloc + l) * nf + e % nf] = acc[b][v];
      }
    }
    if constexpr (EC)
#pragma unroll
      for (int v = 0; v < 4; ++v)   // nodes 16 rb + 4 v ..: function l%16 of E, node l/16
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (two || b == 0)
            hc[b / 2][b % 2] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                acc[b / 2][v], Cs[b % 2][16 * rb + 4 * v + lk][li], hc[b / 2][b % 2], 0, 0, 0);
  }
  if constexpr (EC) {
    if (wave < RB)
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (two || b == 0)
            atomicAdd(&Hs[16 * (b / 2) + 4 * v + lk][16 * (b % 2) + li], hc[b / 2][b % 2][v]);
    __syncthreads();
    for (int i = threadIdx.x; i < ne * ne; i += 512) {
      const int f = i / ne, h = i % ne;
      atomicAdd(&Hee[((int64_t)atom[epair[p0 + f / nf]] * nf + f % nf) * n_enr +
                     (int64_t)atom[epair[p0 + h / nf]] * nf + h % nf],
                -Hs[f][h]);
    }
  }
}

// Rows of the enrichment block of the orthogonalized Hamiltonian, H^E_ee =
// H^phiphi - C B^T - E C^T (the expansion of T^T Hhat T with E = B - C H^cc; the
// projectors' P~^T D P~ is in Hpp already), first part: Hee = H^phiphi
// (symmetrized) - C B^T, row f = (I, k) summed over the support nodes of atom I
// and, at each node, the atoms whose support holds it (B vanishes off the
// support).  C B^T cancels nearly all of H^phiphi and what is left is magnified by
// (M~^ee)^-1, so a filter's output follows the rounding of this sum: over boxes of
// nodes (couple.hip) it takes 3.3 ms instead of 14.1 for 64 atoms, but moves the
// output of degree 40 by 1.5e-9.
__global__ __launch_bounds__(256) void k_hee_rows(int nf, int64_t n_enr,
                                                  const int32_t *__restrict__ snode_ptr,
                                                  const int32_t *__restrict__ snode,
                                                  const int32_t *__restrict__ nm_ptr,
                                                  const int32_t *__restrict__ nm_atom,
                                                  const int32_t *__restrict__ nm_src,
                                                  const double *__restrict__ C_am,
                                                  const double *__restrict__ B_am,
                                                  const double *__restrict__ Hpp,
                                                  double *__restrict__ Hee) {
  extern __shared__ double acc[];
  const int64_t f = blockIdx.x;
  const int I = f / nf, k = f % nf;
  for (int64_t i = threadIdx.x; i < n_enr; i += blockDim.x) acc[i] = 0.0;
  __syncthreads();
  for (int32_t s = snode_ptr[I] + threadIdx.x; s < snode_ptr[I + 1]; s += blockDim.x) {
    const int32_t j = snode[s];
    const double cf = C_am[(int64_t)s * nf + k];
    for (int32_t ee = nm_ptr[j]; ee < nm_ptr[j + 1]; ++ee) {
      const int J = nm_atom[ee];
      const int64_t src = nm_src[ee];
      for (int l = 0; l < nf; ++l) atomicAdd(&acc[J * nf + l], cf * B_am[src * nf + l]);
    }
  }
  __syncthreads();
  for (int64_t i = threadIdx.x; i < n_enr; i += blockDim.x)
    Hee[f * n_enr + i] = 0.5 * (Hpp[f * n_enr + i] + Hpp[i * n_enr + f]) - acc[i];
}

// Projector rows in the orthogonalized basis: P~^phi = P^phi - P^C C^T
// (beta . (phi - C N^C)), one work-group per projector.
__global__ __launch_bounds__(256) void k_ptilde(int nf, int64_t n_enr,
                                                const int32_t *__restrict__ kbnode_ptr,
                                                const int32_t *__restrict__ kbnode,
                                                const double *__restrict__ Pc_am,
                                                const int32_t *__restrict__ nm_ptr,
                                                const int32_t *__restrict__ nm_atom,
                                                const int32_t *__restrict__ nm_src,
                                                const double *__restrict__ C_am,
                                                const double *__restrict__ Pphi,
                                                double *__restrict__ Pt) {
  extern __shared__ double acc[];
  const int K = blockIdx.x;
  for (int64_t i = threadIdx.x; i < n_enr; i += blockDim.x) acc[i] = 0.0;
  __syncthreads();
  for (int32_t s = kbnode_ptr[K] + threadIdx.x; s < kbnode_ptr[K + 1]; s += blockDim.x) {
    const int32_t j = kbnode[s];
    const double pc = Pc_am[s];
    for (int32_t ee = nm_ptr[j]; ee < nm_ptr[j + 1]; ++ee) {
      const int J = nm_atom[ee];
      const int64_t src = nm_src[ee];
      for (int l = 0; l < nf; ++l) atomicAdd(&acc[J * nf + l], pc * C_am[src * nf + l]);
    }
  }
  __syncthreads();
  for (int64_t i = threadIdx.x; i < n_enr; i += blockDim.x)
    Pt[(int64_t)K * n_enr + i] = Pphi[(int64_t)K * n_enr + i] - acc[i];
}

// Symmetrize a square matrix in place: A = (A + A^T)/2
__global__ void k_symmetrize(int64_t n, double *__restrict__ A) {
  int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= n * n) return;
  int64_t i = idx / n, j = idx % n;
  if (j <= i) return;
  double v = 0.5 * (A[i * n + j] + A[j * n + i]);
  A[i * n + j] = v;
  A[j * n + i] = v;
}

// Inverse of each atom-diagonal nf x nf block of M^ee (Gauss-Jordan, pivoted).
__global__ void k_block_inv(int natoms, int nf, int64_t n_enr, const double *__restrict__ Mee,
                            double *__restrict__ inv, int *__restrict__ fail) {
  int I = blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= natoms) return;
  double a[9][18];
  for (int i = 0; i < nf; ++i)
    for (int j = 0; j < nf; ++j) {
      a[i][j] = Mee[(int64_t)(I * nf + i) * n_enr + I * nf + j];
      a[i][nf + j] = (i == j) ? 1.0 : 0.0;
    }
  for (int c = 0; c < nf; ++c) {
    int piv = c;
    for (int r = c + 1; r < nf; ++r)
      if (fabs(a[r][c]) > fabs(a[piv][c])) piv = r;
    if (!(fabs(a[piv][c]) > 0.0)) {
      *fail = 1;
      return;
    }
    if (piv != c)
      for (int j = 0; j < 2 * nf; ++j) {
        double t = a[c][j];
        a[c][j] = a[piv][j];
        a[piv][j] = t;
      }
    double d = 1.0 / a[c][c];
    for (int j = 0; j < 2 * nf; ++j) a[c][j] *= d;
    for (int r = 0; r < nf; ++r)
      if (r != c) {
        double f = a[r][c];
        for (int j = 0; j < 2 * nf; ++j) a[r][j] -= f * a[c][j];
      }
  }
  for (int i = 0; i < nf; ++i)
    for (int j = 0; j < nf; ++j) inv[((int64_t)I * nf + i) * nf + j] = a[i][nf + j];
}

// amp[I] = ||M^phiphi_II||_F ||(M^ee_II)^-1||_F
__global__ void k_block_amp(int natoms, int nf, int64_t n_enr, const double *__restrict__ Mpp,
                            const double *__restrict__ inv, double *__restrict__ amp) {
  const int I = blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= natoms) return;
  double a = 0.0, b = 0.0;
  for (int i = 0; i < nf; ++i)
    for (int j = 0; j < nf; ++j) {
      const double m = Mpp[(int64_t)(I * nf + i) * n_enr + I * nf + j];
      const double v = inv[((int64_t)I * nf + i) * nf + j];
      a += m * m;
      b += v * v;
    }
  amp[I] = sqrt(a) * sqrt(b);
}

// Projector: P^C[s] += sum_q W beta N_l (one block per (atom, cell) pair)
__global__ __launch_bounds__(256) void k_kb_pc(MeshGeo g, double w, double rcut,
                                               const double *__restrict__ xq1,
                                               const double *__restrict__ W3,
                                               const double *__restrict__ N3,
                                               const double *__restrict__ xyz,
                                               const int32_t *__restrict__ pair_atom,
                                               const int32_t *__restrict__ pair_cell,
                                               const int32_t *__restrict__ lmap,
                                               double *__restrict__ Pc) {
  __shared__ double sb[EFE_MAXQ * EFE_MAXQ * EFE_MAXQ];
  const int pr = blockIdx.x;
  const int I = pair_atom[pr], cell = pair_cell[pr];
  for (int q = threadIdx.x; q < g.nqp; q += blockDim.x) {
    double x[3];
    quad_point(g, xq1, cell, q, x);
    double dx = x[0] - xyz[3 * I], dy = x[1] - xyz[3 * I + 1], dz = x[2] - xyz[3 * I + 2];
    sb[q] = W3[q] * kb_beta(dx * dx + dy * dy + dz * dz, w, rcut);
  }
  __syncthreads();
  for (int l = threadIdx.x; l < g.nloc; l += blockDim.x) {
    const int32_t s = lmap[(int64_t)pr * g.nloc + l];
    if (s < 0) continue;
    double acc = 0.0;
    for (int q = 0; q < g.nqp; ++q) acc += sb[q] * N3[(int64_t)q * g.nloc + l];
    atomicAdd(&Pc[s], acc);
  }
}

// Projector-enrichment overlap: Pphi[I][J nf + l] += sum_q W beta_I phi_Jl
__global__ __launch_bounds__(256) void k_kb_pphi(MeshGeo g, EnrParam e, double w, double rcut,
                                                 const double *__restrict__ xq1,
                                                 const double *__restrict__ W3,
                                                 const double *__restrict__ xyz,
                                                 const double *__restrict__ nu,
                                                 const int32_t *__restrict__ trip, int64_t n_enr,
                                                 double *__restrict__ Pphi) {
  __shared__ double red[256][9];
  const int64_t t = blockIdx.x;
  const int cell = trip[3 * t], I = trip[3 * t + 1], J = trip[3 * t + 2];
  double acc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int q = threadIdx.x; q < g.nqp; q += blockDim.x) {
    double x[3], phi[9];
    quad_point(g, xq1, cell, q, x);
    double dx = x[0] - xyz[3 * I], dy = x[1] - xyz[3 * I + 1], dz = x[2] - xyz[3 * I + 2];
    const double b = W3[q] * kb_beta(dx * dx + dy * dy + dz * dz, w, rcut);
    enr_eval(e, x[0] - xyz[3 * J], x[1] - xyz[3 * J + 1], x[2] - xyz[3 * J + 2], phi, nullptr);
    for (int k = 0; k < e.nf; ++k) acc[k] += b * phi[k];
  }
  for (int k = 0; k < 9; ++k) red[threadIdx.x][k] = acc[k];
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s)
      for (int k = 0; k < 9; ++k) red[threadIdx.x][k] += red[threadIdx.x + s][k];
    __syncthreads();
  }
  if (threadIdx.x < (unsigned)e.nf)
    atomicAdd(&Pphi[(int64_t)I * n_enr + J * e.nf + threadIdx.x],
              red[0][threadIdx.x] * nu[J * e.nf + threadIdx.x]);
}

// BF16 operand tiles of v_mfma_f32_16x16x32_bf16 from the FP64 tiles:
// out[cell][rb][ks32][lane][e] = H[16 rb + lane%16][32 ks32 + 8 (lane/16) + e]
__global__ void k_tile_bf16(int64_t n_cells, int RB, int KS, int KS32,
                            const double *__restrict__ H64, uint16_t *__restrict__ out) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t total = n_cells * RB * KS32 * 64 * 8;
  if (idx >= total) return;
  const int e = idx % 8;
  const int lane = (idx / 8) % 64;
  const int ks32 = (idx / 512) % KS32;
  const int64_t crb = idx / (512 * (int64_t)KS32);      // cell * RB + rb
  const int i = lane % 16;
  const int k = 32 * ks32 + 8 * (lane / 16) + e;
  double v = 0.0;
  if (k < 4 * KS) v = H64[(crb * KS + k / 4) * 64 + i + 16 * (k % 4)];
  const __bf16 hb = (__bf16)(float)v;
  out[idx] = *(const uint16_t *)&hb;
}

__global__ void k_fill(int64_t n, double v, double *__restrict__ x) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) x[i] = v;
}

__global__ void k_copy(int64_t n, const double *__restrict__ a, double *__restrict__ b) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) b[i] = a[i];
}

// three copies in one launch
__global__ void k_copy3(int64_t n0, const double *__restrict__ a0, double *__restrict__ b0,
                        int64_t n1, const double *__restrict__ a1, double *__restrict__ b1,
                        int64_t n2, const double *__restrict__ a2, double *__restrict__ b2) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n0) {
    b0[i] = a0[i];
  } else if ((i -= n0) < n1) {
    b1[i] = a1[i];
  } else if ((i -= n1) < n2) {
    b2[i] = a2[i];
  }
}

// Local pseudopotential at every Gauss point: sum_I -Z erf(r/rc)/r + A exp(-(r/rg)^2)
__global__ void k_local_potential(MeshGeo g, const double *__restrict__ xq1, int natoms,
                                  const double *__restrict__ xyz, const double *__restrict__ Z,
                                  double rc, double amp, double rg, double *__restrict__ vq) {
  int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t nq = (int64_t)g.ncell[0] * g.ncell[1] * g.ncell[2] * g.nqp;
  if (idx >= nq) return;
  double x[3];
  quad_point(g, xq1, (int)(idx / g.nqp), (int)(idx % g.nqp), x);
  double v = 0.0;
  for (int I = 0; I < natoms; ++I) {
    double dx = x[0] - xyz[3 * I], dy = x[1] - xyz[3 * I + 1], dz = x[2] - xyz[3 * I + 2];
    double r = sqrt(dx * dx + dy * dy + dz * dz);
    double s = r / rc;
    double eor = s < 1e-6 ? (2.0 / (rc * sqrt(M_PI))) * (1.0 - s * s / 3.0) : erf(s) / r;
    v += -Z[I] * eor + amp * exp(-(r / rg) * (r / rg));
  }
  vq[idx] = v;
}

// Cell Hamiltonians H_c = 1/2 K + N^T diag(w v_c) N (Eq. Hcell with the
// local potential at the Gauss points) on v_mfma_f64_16x16x4.  One work-group
// per (cell, 16-row block): the block's 16 columns of diag(w v_c) N sit in LDS,
// and each wave forms 16 x 16 tiles of the transposed product
// D'[j][i] = sum_q N[q][j] (w v N)[q][16 rb + i], whose accumulator layout
// (lane l of register v: j = j0 + 4 v + l/16, i = l % 16) is exactly the
// stored operand layout tile[cell][rb][j/4][i + 16 (j%4)] = base + 16 j + i,
// so every register is one contiguous 512-byte store.  Quadrature steps past
// nqp meet zero rows of the LDS strip.
typedef double v4d_b __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void k_build_hcell(int nloc, int nqp, int RB, int KS, int KQ8,
                                                     const double *__restrict__ N3,
                                                     const double *__restrict__ W3,
                                                     const double *__restrict__ K,
                                                     const double *__restrict__ vq,
                                                     double *__restrict__ H64,
                                                     float *__restrict__ H32) {
  extern __shared__ double bs[];   // [4 KQ8][16]: (w v N)[q][16 rb + i]
  const int cell = blockIdx.x / RB, rb = blockIdx.x % RB;
  for (int idx = threadIdx.x; idx < 64 * KQ8; idx += blockDim.x) {
    const int q = idx / 16, row = 16 * rb + idx % 16;
    bs[idx] = (q < nqp && row < nloc)
                  ? W3[q] * vq[(int64_t)cell * nqp + q] * N3[(int64_t)q * nloc + row]
                  : 0.0;
  }
  __syncthreads();
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, li = lane % 16, lk = lane / 16;
  const int JT = (4 * KS + 15) / 16;
  const int64_t tbase = ((int64_t)cell * RB + rb) * KS * 64;
  for (int jt = wave; jt < JT; jt += 4) {
    const int j0 = 16 * jt;
    const double *np = N3 + min(j0 + li, nloc - 1);
    v4d_b acc = {0.0, 0.0, 0.0, 0.0};
    double a[8], na[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) a[s] = np[(int64_t)min(4 * s + lk, nqp - 1) * nloc];
    for (int k0 = 0; k0 < KQ8; k0 += 8) {
      // next batch of N^T fragments (clamped rows; they meet zero LDS rows)
#pragma unroll
      for (int s = 0; s < 8; ++s)
        na[s] = np[(int64_t)min(4 * (k0 + 8 + s) + lk, nqp - 1) * nloc];
#pragma unroll
      for (int s = 0; s < 8; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], bs[(4 * (k0 + s) + lk) * 16 + li], acc,
                                                   0, 0, 0);
#pragma unroll
      for (int s = 0; s < 8; ++s) a[s] = na[s];
    }
    const int row = 16 * rb + li;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = j0 + 4 * v + lk;
      if (j >= 4 * KS) continue;
      const double h =
          (row < nloc && j < nloc) ? 0.5 * K[(int64_t)row * nloc + j] + acc[v] : 0.0;
      H64[tbase + 16 * j + li] = h;
      if (H32) H32[tbase + 16 * j + li] = (float)h;
    }
  }
}

// ------------------------------------------------------------ host launchers
efe_status efe_build_reference(efe_ctx *c) {
  std::vector<double> xg, wg, xq, wq;
  gll_rule(c->p, xg, wg);
  gauss_rule(c->nq, xq, wq);
  std::vector<double> N1, D1;
  lagrange(xg, xq, N1, D1);
  double *dN1, *dD1, *dwq, *dwg;
  efe_status s;
  if ((s = efe_alloc(c, (void **)&dN1, N1.size() * 8))) return s;
  if ((s = efe_alloc(c, (void **)&dD1, D1.size() * 8))) return s;
  if ((s = efe_alloc(c, (void **)&dwq, wq.size() * 8))) return s;
  if ((s = efe_alloc(c, (void **)&dwg, wg.size() * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_xq1, xq.size() * 8))) return s;
  HIPCHK(c, hipMemcpyAsync(dN1, N1.data(), N1.size() * 8, hipMemcpyHostToDevice, c->stream));
  HIPCHK(c, hipMemcpyAsync(dD1, D1.data(), D1.size() * 8, hipMemcpyHostToDevice, c->stream));
  HIPCHK(c, hipMemcpyAsync(dwq, wq.data(), wq.size() * 8, hipMemcpyHostToDevice, c->stream));
  HIPCHK(c, hipMemcpyAsync(dwg, wg.data(), wg.size() * 8, hipMemcpyHostToDevice, c->stream));
  HIPCHK(c, hipMemcpyAsync(c->d_xq1, xq.data(), xq.size() * 8, hipMemcpyHostToDevice, c->stream));
  const int64_t nt = (int64_t)c->nqp * c->nloc;
  if ((s = efe_alloc(c, (void **)&c->d_N3, nt * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_G3, 3 * nt * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_W3, c->nqp * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_K, (int64_t)c->nloc * c->nloc * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_m, c->n_nodes * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_minv, c->n_nodes * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_m_int, c->n_nodes * 8))) return s;
  k_ref3d<<<cdiv(nt, 256), 256, 0, c->stream>>>(c->P, c->nq, dN1, dD1, dwq, c->h[0], c->h[1],
                                                c->h[2], c->d_N3, c->d_G3, c->d_W3);
  k_stiffness<<<cdiv((int64_t)c->nloc * c->nloc, 256), 256, 0, c->stream>>>(c->nloc, c->nqp,
                                                                             c->d_G3, c->d_W3, c->d_K);
  k_lumped_mass<<<cdiv(c->n_nodes, 256), 256, 0, c->stream>>>(
      c->n1[0], c->n1[1], c->n1[2], c->p, dwg, c->h[0], c->h[1], c->h[2], c->d_m, c->d_minv, c->d_m_int);
  HIPCHK(c, hipGetLastError());
  HIPCHK(c, hipStreamSynchronize(c->stream));
  efe_free(c, dN1);
  efe_free(c, dD1);
  efe_free(c, dwq);
  efe_free(c, dwg);
  // MFMA tile geometry of the dense cell products
  c->KP = (int)cdiv(c->nloc, 4) * 4;
  c->KS = c->KP / 4;
  c->RB = (int)cdiv(c->nloc, 16);
  c->KS32 = (int)cdiv(c->nloc, 32);
  std::vector<long double> xgl, wgl, xql, wql, N1l, D1l, Il, Dl;
  gll_rule(c->p, xgl, wgl);
  gauss_rule(c->nq, xql, wql);
  lagrange(xgl, xql, N1l, D1l);
  lagrange(xql, xql, Il, Dl);
  return efe_tp_setup(c, wq, N1, D1, wg, wql, N1l, Dl);
}

efe_status efe_build_enrichment(efe_ctx *c) {
  efe_status s;
  const MeshGeo g = mesh_geo(c);
  const EnrParam e = enr_param(c);
  const int nf = c->nf;
  const int64_t ne = c->n_enr;
  const int64_t ns = c->n_snodes * nf;
  if ((s = efe_alloc(c, (void **)&c->d_nu, ne * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_b_am, ns * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_C_am, ns * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_Bkin_am, ns * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_B_am, ns * 8))) return s;
  const int64_t ng = c->n_gslots * nf * 8;
  if ((s = efe_alloc(c, (void **)&c->d_Cg, ng * 8))) return s;
  if (ng) {
    HIPCHK(c, hipMemsetAsync(c->d_Cg, 0, ng * 8, c->stream));
  }
  if ((s = efe_alloc(c, (void **)&c->d_Mpp, ne * ne * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_Mee, ne * ne * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_Hpp_kin, ne * ne * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_Hpp, ne * ne * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_Mee_inv, (int64_t)c->natoms * nf * nf * 8))) return s;
  HIPCHK(c, hipMemsetAsync(c->d_nu, 0, ne * 8, c->stream));
  HIPCHK(c, hipMemsetAsync(c->d_b_am, 0, ns * 8, c->stream));
  HIPCHK(c, hipMemsetAsync(c->d_Bkin_am, 0, ns * 8, c->stream));
  HIPCHK(c, hipMemsetAsync(c->d_Mpp, 0, ne * ne * 8, c->stream));
  HIPCHK(c, hipMemsetAsync(c->d_Hpp_kin, 0, ne * ne * 8, c->stream));
  if (nf > 0 && c->npairs > 0) {
    k_enr_norm<<<c->npairs, 256, 0, c->stream>>>(g, e, c->d_xq1, c->d_W3, c->d_xyz,
                                                 c->d_pair_atom, c->d_pair_cell, c->d_nu);
    k_inv_sqrt<<<cdiv(ne, 256), 256, 0, c->stream>>>(ne, c->d_nu);
    if ((s = efe_alloc(c, (void **)&c->d_Bkin_pair, (size_t)c->npairs * c->nloc * nf * 8)))
      return s;
    k_enr_pair_proj<true><<<c->npairs, 256, 0, c->stream>>>(
        g, e, c->d_xq1, c->d_W3, c->d_N3, c->d_G3, c->d_xyz, c->d_nu, c->d_pair_atom,
        c->d_pair_cell, c->d_pair_lmap, nullptr, c->d_b_am, c->d_Bkin_am, c->d_Bkin_pair);
    k_scale_by_minv<<<cdiv(ns, 256), 256, 0, c->stream>>>(c->n_snodes, nf, c->d_snode, c->d_minv,
                                                          c->d_b_am, c->d_C_am);
    k_to_group_major<<<cdiv(c->n_nodes, 256), 256, 0, c->stream>>>(
        c->n_nodes, nf, c->d_nm_ptr, c->d_nm_src, c->d_nm_gslot, c->d_C_am, c->d_Cg);
    if (c->ntrip > 0)
      k_enr_pp<<<c->ntrip, 128, 0, c->stream>>>(g, e, c->d_xq1, c->d_W3, c->d_xyz, c->d_nu,
                                                      c->d_trip, ne, c->d_Mpp,
                                                      c->d_Hpp_kin);
    k_symmetrize<<<cdiv(ne * ne, 256), 256, 0, c->stream>>>(ne, c->d_Mpp);
    k_symmetrize<<<cdiv(ne * ne, 256), 256, 0, c->stream>>>(ne, c->d_Hpp_kin);
    if (ne * 8 > 150 * 1024) EFE_FAIL(c, EFE_EINVAL, "too many enrichment functions for M^ee rows");
    k_mee_rows<<<ne, 256, ne * 8, c->stream>>>(nf, ne, c->d_snode_ptr, c->d_snode, c->d_nm_ptr,
                                               c->d_nm_atom, c->d_nm_src, c->d_C_am, c->d_b_am,
                                               c->d_Mpp, c->d_Mee);
    k_symmetrize<<<cdiv(ne * ne, 256), 256, 0, c->stream>>>(ne, c->d_Mee);
    int *dfail;
    if ((s = efe_alloc(c, (void **)&dfail, sizeof(int)))) return s;
    HIPCHK(c, hipMemsetAsync(dfail, 0, sizeof(int), c->stream));
    k_block_inv<<<cdiv(c->natoms, 64), 64, 0, c->stream>>>(c->natoms, nf, ne, c->d_Mee,
                                                           c->d_Mee_inv, dfail);
    int hfail = 0;
    HIPCHK(c, hipMemcpyAsync(&hfail, dfail, sizeof(int), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    efe_free(c, dfail);
    if (hfail) EFE_FAIL(c, EFE_ENUMERIC, "singular atom block of M^ee");
    double *damp;
    if ((s = efe_alloc(c, (void **)&damp, (size_t)c->natoms * 8))) return s;
    k_block_amp<<<cdiv(c->natoms, 64), 64, 0, c->stream>>>(c->natoms, nf, ne, c->d_Mpp,
                                                           c->d_Mee_inv, damp);
    std::vector<double> amp(c->natoms);
    HIPCHK(c, hipMemcpyAsync(amp.data(), damp, (size_t)c->natoms * 8, hipMemcpyDeviceToHost,
                             c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    efe_free(c, damp);
    c->amplification = 1.0;
    for (double a : amp) c->amplification = std::max(c->amplification, a);
  }
  // projectors
  const int np = c->nproj;
  if ((s = efe_alloc(c, (void **)&c->d_Pc_am, c->n_kbnodes * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_Pphi, (int64_t)np * ne * 8))) return s;
  if ((s = efe_alloc(c, (void **)&c->d_D, np * 8))) return s;
  HIPCHK(c, hipMemsetAsync(c->d_Pc_am, 0, c->n_kbnodes * 8, c->stream));
  HIPCHK(c, hipMemsetAsync(c->d_Pphi, 0, (int64_t)np * ne * 8, c->stream));
  if (np > 0) {
    k_fill<<<cdiv(np, 256), 256, 0, c->stream>>>(np, c->kb_D, c->d_D);
    k_kb_pc<<<c->nkbpairs, 256, 0, c->stream>>>(g, c->kb_width, c->kb_rcut, c->d_xq1, c->d_W3,
                                                c->d_N3, c->d_xyz, c->d_kbpair_atom,
                                                c->d_kbpair_cell, c->d_kbpair_lmap, c->d_Pc_am);
    if (c->nkbtrip > 0)
      k_kb_pphi<<<c->nkbtrip, 256, 0, c->stream>>>(g, e, c->kb_width, c->kb_rcut, c->d_xq1,
                                                   c->d_W3, c->d_xyz, c->d_nu, c->d_kbtrip, ne,
                                                   c->d_Pphi);
  }
  // projector rows in the orthogonalized basis
  if ((s = efe_alloc(c, (void **)&c->d_Ptil, (int64_t)np * ne * 8))) return s;
  if (np > 0 && ne > 0)
    k_ptilde<<<np, 256, ne * 8, c->stream>>>(nf, ne, c->d_kbnode_ptr, c->d_kbnode, c->d_Pc_am,
                                             c->d_nm_ptr, c->d_nm_atom, c->d_nm_src, c->d_C_am,
                                             c->d_Pphi, c->d_Ptil);
  HIPCHK(c, hipGetLastError());
  // the projectors' part P~^T D P~ of H^E_ee does not depend on the potential
  if (np > 0 && ne > 0 &&
      (s = efe_dgemm(c, true, false, ne, ne, np, 1.0, c->d_Ptil, ne, c->d_Ptil, ne, 1.0,
                     c->d_Hpp_kin, ne, c->d_D)))
    return s;
  return efe_couple_projectors(c);
}

efe_status efe_launch_local_potential(efe_ctx *c, double *vq) {
  const MeshGeo g = mesh_geo(c);
  k_local_potential<<<cdiv(c->n_qpts, 256), 256, 0, c->stream>>>(
      g, c->d_xq1, c->natoms, c->d_xyz, c->d_Zs, c->loc_rc, c->loc_amp, c->loc_rg, vq);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}

efe_status efe_build_operators(efe_ctx *c, const double *vq, int precisions) {
  efe_status s;
  struct Building {   // until the call returns
    efe_ctx *c;
    explicit Building(efe_ctx *x) : c(x) { c->building = true; }
    ~Building() { c->building = false; }
  } building(c);
  c->ws_refused = SIZE_MAX;
  const MeshGeo g = mesh_geo(c);
  const EnrParam e = enr_param(c);
  const int nf = c->nf;
  const int64_t ne = c->n_enr;
  const int64_t tiles = c->n_cells * c->RB * c->KS * 64;
  // every allocation before the first launch: a call that fails for memory
  // leaves the operators of the potential before it whole
  if (!c->d_vq && (s = efe_alloc(c, (void **)&c->d_vq, c->n_qpts * 8))) return s;
  const bool want32 = precisions & (1 << EFE_FP32);
  const bool want16 = precisions & (1 << EFE_BF16);
  // dense cell Hamiltonians: for E_c, and where an apply takes them (Gauss rules
  // without tensor products, and the BF16 copies)
  const bool coupled = nf > 0 && c->npairs > 0;
  const bool dense = !c->tp || want16 || coupled;
  if (dense && !c->d_Htile64 && (s = efe_alloc(c, (void **)&c->d_Htile64, tiles * 8))) return s;
  if (want32 && !c->tp && !c->d_Htile32 && (s = efe_alloc(c, (void **)&c->d_Htile32, tiles * 4))) return s;
  const int64_t tiles16 = c->n_cells * c->RB * c->KS32 * 64 * 8;
  if (want16 && !c->d_Htile16 && (s = efe_alloc(c, (void **)&c->d_Htile16, tiles16 * 2))) return s;
  const int KQ8 = (int)cdiv(cdiv(c->nqp, 4), 8) * 8;   // quadrature k steps, padded
  const size_t shm = (size_t)KQ8 * 64 * 8;
  if (shm > 64 * 1024) EFE_FAIL(c, EFE_EINVAL, "too many Gauss points per cell");
  if (coupled) {
    const size_t pb = (size_t)c->npairs * c->nloc * nf * 8;   // support pairs
    if (!c->d_B_pair && (s = efe_alloc(c, (void **)&c->d_B_pair, pb))) return s;
    if (!c->d_Epair && (s = efe_alloc(c, (void **)&c->d_Epair, (size_t)c->ncpairs * c->nloc * nf * 8)))
      return s;
  }
  if (ne && !c->d_Hee && (s = efe_alloc(c, (void **)&c->d_Hee, ne * ne * 8))) return s;
  if ((s = efe_couple_alloc(c, want32))) return s;
  // the potential, and what it adds to: the kinetic parts of B and H^phiphi
  const int64_t ns = coupled ? c->n_snodes * nf : 0, ns2 = coupled ? ne * ne : 0;
  k_copy3<<<cdiv(c->n_qpts + ns + ns2, 256), 256, 0, c->stream>>>(
      c->n_qpts, vq, c->d_vq, ns, c->d_Bkin_am, c->d_B_am, ns2, c->d_Hpp_kin, c->d_Hpp);
  if (dense)
    k_build_hcell<<<c->n_cells * c->RB, 256, shm, c->stream>>>(
        c->nloc, c->nqp, c->RB, c->KS, KQ8, c->d_N3, c->d_W3, c->d_K, c->d_vq, c->d_Htile64,
        want32 && !c->tp ? c->d_Htile32 : nullptr);
  if (want16)
    k_tile_bf16<<<cdiv(tiles16, 256), 256, 0, c->stream>>>(c->n_cells, c->RB, c->KS, c->KS32,
                                                           c->d_Htile64, c->d_Htile16);
  c->have32 = want32;
  c->have16 = want16;
  if (coupled) {
    const int KQ = (int)cdiv(c->nqp, 4);
#define GO(P)                                                                                  \
  k_enr_pair_proj_tp<P><<<c->npairs, PAIR_TP_T, 0, c->stream>>>(                               \
      g, e, c->d_xq1, c->d_W3, c->d_tpm, c->d_xyz, c->d_nu, c->d_pair_atom, c->d_pair_cell,    \
      c->d_pair_lmap, c->d_vq, c->d_B_am, c->d_Bkin_pair, c->d_B_pair)
    switch (c->tp ? c->P : 0) {
      case 2: GO(2); break;
      case 3: GO(3); break;
      case 4: GO(4); break;
      case 5: GO(5); break;
      case 6: GO(6); break;
      case 7: GO(7); break;
      default:
        k_enr_pair_proj_v<<<c->npairs, 256, (size_t)KQ * 64 * 8, c->stream>>>(
            g, e, c->d_xq1, c->d_W3, c->d_N3, c->d_xyz, c->d_nu, c->d_pair_atom, c->d_pair_cell,
            c->d_pair_lmap, c->d_vq, KQ, c->d_B_am, c->d_Bkin_pair, c->d_B_pair);
    }
#undef GO
    if (c->n_ppv > 0)
      k_enr_ppv<<<c->n_ppv, 256, 0, c->stream>>>(g, e, c->d_xq1, c->d_W3, c->d_xyz, c->d_nu,
                                                c->d_ppv, c->d_trip, c->d_vq, ne, c->d_Hpp);
    k_hee_rows<<<ne, 256, ne * 8, c->stream>>>(nf, ne, c->d_snode_ptr, c->d_snode, c->d_nm_ptr,
                                               c->d_nm_atom, c->d_nm_src, c->d_C_am, c->d_B_am,
                                               c->d_Hpp, c->d_Hee);
    // coupling of the orthogonalized basis, E_c per (atom, cell) pair
    const int mcb = (int)cdiv(c->max_rbe, 2);
    const int64_t nwg = cdiv(c->n_cells, 8) * 8 * mcb;
#define GO(EC)                                                                                    \
  k_build_E<EC><<<nwg, 512, 0, c->stream>>>(                                                      \
      c->n_cells, c->nloc, c->RB, c->KS, nf, mcb, c->d_Htile64, c->d_cell_eptr, c->d_cell_epair,  \
      c->d_cpair_lmap, c->d_cpair_spair, c->d_C_am, c->d_B_pair, c->d_Epair, c->d_cpair_atom, ne, \
      c->d_Hee)
    if (c->max_rbe <= 2)
      GO(true);
    else
      GO(false);
#undef GO
  } else if (ne) {
    k_copy<<<cdiv(ne * ne, 256), 256, 0, c->stream>>>(ne * ne, c->d_Hpp_kin, c->d_Hee);
  }
  if ((s = efe_couple_build(c, want32))) return s;
  HIPCHK(c, hipGetLastError());
  c->have_potential = true;
  return EFE_OK;
}
