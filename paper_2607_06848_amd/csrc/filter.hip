// Chebyshev filtering (Sec. III.B) and the Lanczos spectrum bound.
//
// Residual filter (Eqs. residual, residualapprox, with the coefficients that
// follow from inserting Eq. ChebyRecur into the definition of Z_k):
//   G   = H V - M V Lambda
//   Z_1 = (s_1/e) G,  Z_0 = 0
//   Z_k = (2 s_k/e) H M~^-1 Z_{k-1} - (2 c s_k/e) Z_{k-1} - s_{k-1} s_k Z_{k-2}
//         + (2 s_k/e) G C_{k-1}(Lambda)
//   V  <- M~^-1 Z_m + V C_m(Lambda)
// M~^-1 is folded into the H apply: its CFE part (1/m) into the reading of the
// rows, its enrichment part (nf x nf blocks) into the coefficients.  Z_k overwrites Z_{k-2}.
#include <cmath>
#include <vector>

#include "efe_device.h"

// sigma_1 = e / (a_min - c), sigma_k = 1 / (2 / sigma_1 - sigma_{k-1})
__global__ void k_sigma_table(int m, double a, double b, double a_min, double *__restrict__ sig) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double cc = 0.5 * (a + b), e = 0.5 * (b - a);
  sig[0] = 0.0;
  sig[1] = e / (a_min - cc);
  for (int k = 2; k <= m; ++k) sig[k] = 1.0 / (2.0 / sig[1] - sig[k - 1]);
}

// C_k(lambda_j), k = 0..m, by the scalar recurrence (one thread per column)
__global__ void k_cheb_table(int m, int ncols, const double *__restrict__ lam, double c, double e,
                             const double *__restrict__ sig, double *__restrict__ T) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= ncols) return;
  const double x = lam[j];
  double cm2 = 1.0, cm1 = sig[1] * (x - c) / e;
  T[j] = 1.0;
  if (m >= 1) T[ncols + j] = cm1;
  for (int k = 2; k <= m; ++k) {
    const double ck = (2.0 * sig[k] / e) * (x - c) * cm1 - sig[k - 1] * sig[k] * cm2;
    T[(int64_t)k * ncols + j] = ck;
    cm2 = cm1;
    cm1 = ck;
  }
}

// G = W - MV diag(lam) over all rows (ld of G, W, MV = ncols); Z = s G
// (MV and Zp may be the same buffer)
__global__ void k_residual_init(int64_t rows, int ncols, const double *__restrict__ W,
                                const double *MV, const double *__restrict__ lam, double s1e,
                                double *__restrict__ G, double *__restrict__ Z, double *Zp) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= rows * ncols) return;
  const double mv = MV[idx];
  const double g = W[idx] - mv * lam[idx % ncols];
  G[idx] = g;
  Z[idx] = s1e * g;
  Zp[idx] = 0.0;
}

// V <- w_r Z + V Cl on CFE rows (w = 1/m), enrichment rows use ZE = M~ee^-1 Z^E
__global__ void k_vout(int64_t n_nodes, int64_t rows, int ncols, const double *__restrict__ minv,
                       const double *__restrict__ Z, const double *__restrict__ ZE,
                       const double *__restrict__ Cl, double *__restrict__ V, int64_t ld) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= rows * ncols) return;
  const int64_t r = idx / ncols;
  const int j = idx % ncols;
  const double y = r < n_nodes ? minv[r] * Z[idx] : ZE[(r - n_nodes) * ncols + j];
  double v = V[r * ld + j] * Cl[j];
  if (r < n_nodes && minv[r] == 0.0) v = 0.0;
  V[r * ld + j] = y + v;
}

// standard filter step on A = M~^-1 H:
// Yn = a (AY - c Y) + gam Yp with AY = (1/m) W on CFE rows, WE on enrichment rows
__global__ void k_std_step(int64_t n_nodes, int64_t rows, int ncols, double a, double cc,
                           double gam, const double *__restrict__ minv,
                           const double *__restrict__ W, const double *__restrict__ WE,
                           const double *__restrict__ Y, const double *Yp, double *Yn) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= rows * ncols) return;
  const int64_t r = idx / ncols;
  const double ay = r < n_nodes ? minv[r] * W[idx] : WE[idx - n_nodes * ncols];
  const double yp = Yp ? Yp[idx] : 0.0;
  Yn[idx] = a * (ay - cc * Y[idx]) + gam * yp;
}

__global__ void k_copy_in(int64_t rows, int ncols, const double *__restrict__ src, int64_t lds,
                          double *__restrict__ dst, int64_t ldd) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= rows * ncols) return;
  const int64_t r = idx / ncols;
  const int j = idx % ncols;
  dst[r * ldd + j] = src[r * lds + j];
}

// ------------------------------------------------------------------ filter
// One column chunk of the filter (the filter acts on every column on its own,
// so chunks of a wide block give the same result as one pass over it).
static efe_status filter_chunk(efe_ctx *c, double *V, const double *lambda, int32_t ncols,
                               int64_t ld, const efe_cheb_params *prm) {
  efe_status s;
  const int m = prm->degree;
  const double cc = 0.5 * (prm->a + prm->b), e = 0.5 * (prm->b - prm->a);
  std::vector<double> sig(m + 1, 0.0);
  sig[1] = e / (prm->a_min - cc);
  for (int k = 2; k <= m; ++k) sig[k] = 1.0 / (2.0 / sig[1] - sig[k - 1]);
  const int64_t rows = c->rows, nn = c->n_nodes;
  const int64_t blk = rows * ncols;
  double *G, *Za, *Zb, *W, *XE, *Cl, *dsig;
  if ((s = efe_ws(c, 2, blk * 8, (void **)&G))) return s;
  if ((s = efe_ws(c, 3, blk * 8, (void **)&Za))) return s;
  if ((s = efe_ws(c, 4, blk * 8, (void **)&Zb))) return s;
  if ((s = efe_ws(c, 5, blk * 8, (void **)&W))) return s;
  if ((s = efe_ws(c, 6, (size_t)std::max<int64_t>(c->n_enr, 1) * ncols * 8, (void **)&XE))) return s;
  if ((s = efe_ws(c, 7, (size_t)(m + 1) * ncols * 8, (void **)&Cl))) return s;
  if ((s = efe_ws(c, 8, (size_t)(m + 1) * 8, (void **)&dsig))) return s;
  // the same table on the device (the same IEEE operations in the same order
  // as the host's, so both hold identical values)
  k_sigma_table<<<1, 1, 0, c->stream>>>(m, prm->a, prm->b, prm->a_min, dsig);
  const int T = 256;
  const int64_t nb = cdiv(blk, T);

  if (prm->mode == EFE_FILTER_STANDARD) {
    // Y_0 = V (copied to Za), Y_1 = (s1/e)(A V - c V), Y_k = (2 s_k/e)(A - c) Y_{k-1} - s s Y_{k-2}
    k_copy_in<<<nb, T, 0, c->stream>>>(rows, ncols, V, ld, Za, ncols);
    double *Yp = nullptr, *Yc = Za, *Yn = Zb;
    for (int k = 1; k <= m; ++k) {
      if ((s = efe_apply_H_internal(c, Yc, ncols, false, Yc + nn * ncols, ncols, W, ncols, ncols,
                                    prm->prec)))
        return s;
      if ((s = efe_enr_block_inv(c, W + nn * ncols, ncols, XE, ncols, ncols))) return s;
      const double a = (k == 1 ? 1.0 : 2.0) * sig[k] / e;
      const double gam = k == 1 ? 0.0 : -sig[k - 1] * sig[k];
      k_std_step<<<nb, T, 0, c->stream>>>(nn, rows, ncols, a, cc, gam, c->d_minv, W, XE, Yc,
                                          k == 1 ? nullptr : Yp, Yn);
      double *t = Yp ? Yp : G;
      Yp = Yc;
      Yc = Yn;
      Yn = t;
    }
    k_copy_in<<<nb, T, 0, c->stream>>>(rows, ncols, Yc, ncols, V, ld);
    HIPCHK(c, hipGetLastError());
    return EFE_OK;
  }

  k_cheb_table<<<cdiv(ncols, 64), 64, 0, c->stream>>>(m, ncols, lambda, cc, e, dsig, Cl);
  // G = H V - M V Lambda (MV staged in Zb)
  if ((s = efe_apply_H_internal(c, V, ld, false, V + nn * ld, ld, W, ncols, ncols, EFE_FP64)))
    return s;
  if ((s = efe_apply_M_internal(c, V, ld, Zb, ncols, ncols))) return s;
  double *Zc = Za, *Zp = Zb;
  k_residual_init<<<nb, T, 0, c->stream>>>(rows, ncols, W, Zb, lambda, sig[1] / e, G, Zc, Zp);
  for (int k = 2; k <= m; ++k) {
    // the recurrence's H applies run in the requested precision (G stays
    // FP64); its three affine terms are added where alpha H M~^-1 Z_{k-1} is
    // assembled, and Z_k is written in place of Z_{k-2}
    ApplyEpilogue ep;
    ep.alpha = 2.0 * sig[k] / e;
    ep.beta = -cc * ep.alpha;
    ep.gamma = -sig[k - 1] * sig[k];
    ep.Z1 = Zc;
    ep.Z2 = Zp;
    ep.G = G;
    ep.Cl = Cl + (int64_t)(k - 1) * ncols;
    const int t = efe_timer_begin(c, EFE_T_RECUR);
    if ((s = efe_apply_H_internal(c, Zc, ncols, true, Zc + nn * ncols, ncols, Zp, ncols, ncols,
                                  prm->prec, &ep)))
      return s;
    efe_timer_end(c, EFE_T_RECUR, t);
    std::swap(Zc, Zp);
  }
  if ((s = efe_enr_block_inv(c, Zc + nn * ncols, ncols, XE, ncols, ncols))) return s;
  k_vout<<<nb, T, 0, c->stream>>>(nn, rows, ncols, c->d_minv, Zc, XE, Cl + (int64_t)m * ncols, V, ld);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}

efe_status efe_filter_check(efe_ctx *c, double *V, const double *lambda, int32_t ncols,
                            int64_t ld, const efe_cheb_params *prm) {
  if (!c) return EFE_EINVAL;
  if (!V || !prm || ncols < 0 || ld < ncols || ld < 1) EFE_FAIL(c, EFE_EINVAL, "bad arguments");
  if (prm->degree < 1) EFE_FAIL(c, EFE_EINVAL, "degree must be >= 1");
  if (!(prm->a < prm->b) || !(prm->a_min < prm->a)) EFE_FAIL(c, EFE_EINVAL, "need a_min < a < b");
  if (prm->mode != EFE_FILTER_RESIDUAL && prm->mode != EFE_FILTER_STANDARD)
    EFE_FAIL(c, EFE_EINVAL, "bad filter mode");
  if (prm->prec != EFE_FP64 && prm->prec != EFE_FP32 && prm->prec != EFE_BF16)
    EFE_FAIL(c, EFE_EINVAL, "bad filter precision");
  if (prm->mode == EFE_FILTER_RESIDUAL && !lambda) EFE_FAIL(c, EFE_EINVAL, "residual mode needs lambda");
  if (prm->prec == EFE_BF16 && c->amplification > EFE_BF16_MAX_AMPLIFICATION)
    EFE_FAIL(c, EFE_EINVAL,
             "BF16 filter refused: enrichment amplification " + std::to_string(c->amplification) +
                 " exceeds " + std::to_string(EFE_BF16_MAX_AMPLIFICATION));
  if (!c->have_potential) EFE_FAIL(c, EFE_ESTATE, "no potential set");
  return EFE_OK;
}

efe_status efe_filter_run(efe_ctx *c, double *V, const double *lambda, int32_t ncols, int64_t ld,
                          const efe_cheb_params *prm) {
  efe_status s;
  for (int32_t j0 = 0; j0 < ncols; j0 += c->col_chunk) {
    const int32_t nc = std::min<int32_t>(c->col_chunk, ncols - j0);
    if ((s = filter_chunk(c, V + j0, lambda ? lambda + j0 : nullptr, nc, ld, prm))) return s;
  }
  return EFE_OK;
}

extern "C" efe_status efe_cheb_filter(efe_ctx *c, double *V, const double *lambda, int32_t ncols,
                                      int64_t ld, const efe_cheb_params *prm) {
  efe_status s = efe_filter_check(c, V, lambda, ncols, ld, prm);
  if (s) return s;
  return efe_filter_run(c, V, lambda, ncols, ld, prm);
}

// ------------------------------------------------------------------ Lanczos
// Vectors are rows long: CFE rows first, then the enrichment rows of every
// atom.  The inner product is that of M~: m on CFE rows, the atom blocks of
// M^ee on enrichment rows.  Work-groups 0 .. nbc - 1 take CFE rows, the others
// atoms, 16 lanes each (one thread per atom left 50 us of dependent loads).
// Dot products go through LZ_NP per-work-group partial sums, which every
// work-group of the next kernel adds itself in the same order: no atomics, no
// extra launches (one launch per dot product, 231 of them in 20 steps, took
// 7.6 of the 64-atom bound's 16.9 ms).
constexpr int LZ_NP = 512, LZ_T = 256;

__device__ inline double lz_block_sum(double x, double *red) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = x;
  __syncthreads();
  const double s = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return s;
}

// total of one row of partial sums (every thread gets it)
__device__ inline double lz_total(const double *__restrict__ part, double *red) {
  return lz_block_sum(part[threadIdx.x] + part[threadIdx.x + LZ_T], red);
}

struct LzArgs {
  int64_t nn, n_enr;
  int natoms, nf, nbc;
  const double *m, *minv, *Mee, *inv;
};

// loop of a CFE work-group over its rows, and of an atom work-group over its
// atoms: f(I, k) with k the lane's function (every lane of a group runs it)
template <class F>
__device__ inline void lz_rows(const LzArgs &a, F &&f) {
  if ((int)blockIdx.x >= a.nbc) return;
  for (int64_t i = blockIdx.x * (int64_t)LZ_T + threadIdx.x; i < a.nn; i += (int64_t)a.nbc * LZ_T)
    f(i);
}
template <class F>
__device__ inline void lz_atoms(const LzArgs &a, F &&f) {
  if ((int)blockIdx.x < a.nbc) return;
  const int per = LZ_T / 16, g = (int)blockIdx.x - a.nbc, ng = (int)gridDim.x - a.nbc;
  for (int I = g * per + (int)threadIdx.x / 16; I < a.natoms; I += ng * per)
    f(I, (int)threadIdx.x % 16);
}
// (M^ee_II x)_k from the lanes' x (zero in lanes k >= nf)
__device__ inline double lz_block_row(const LzArgs &a, int I, int k, double x) {
  double s = 0.0;
  for (int l = 0; l < a.nf; ++l) {
    const double xl = __shfl(x, l, 16);
    if (k < a.nf) s += a.Mee[((int64_t)I * a.nf + k) * a.n_enr + (int64_t)I * a.nf + l] * xl;
  }
  return s;
}

// y = x without its boundary rows; partial sums of y.M~ y
__global__ __launch_bounds__(LZ_T) void k_lz_start(LzArgs a, const double *__restrict__ x,
                                                   double *__restrict__ y,
                                                   double *__restrict__ part) {
  __shared__ double red[4];
  double s = 0.0;
  lz_rows(a, [&](int64_t i) {
    const double v = a.minv[i] == 0.0 ? 0.0 : x[i];
    y[i] = v;
    s += a.m[i] * v * v;
  });
  lz_atoms(a, [&](int I, int k) {
    const int64_t r = a.nn + (int64_t)I * a.nf + k;
    const double v = k < a.nf ? x[r] : 0.0;
    if (k < a.nf) y[r] = v;
    s += v * lz_block_row(a, I, k, v);
  });
  const double t = lz_block_sum(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// y = x / b with b = sqrt of the summed partials, which is kept in beta_out
__global__ __launch_bounds__(LZ_T) void k_lz_scale(int64_t n, const double *__restrict__ part,
                                                   const double *__restrict__ x,
                                                   double *__restrict__ y,
                                                   double *__restrict__ beta_out) {
  __shared__ double red[4];
  const double b = sqrt(lz_total(part, red));
  if (blockIdx.x == 0 && threadIdx.x == 0 && beta_out) *beta_out = b;
  for (int64_t i = blockIdx.x * (int64_t)LZ_T + threadIdx.x; i < n; i += (int64_t)gridDim.x * LZ_T)
    y[i] = x[i] / b;
}

// partial sums of v.u
__global__ __launch_bounds__(LZ_T) void k_lz_dot(int64_t n, const double *__restrict__ v,
                                                 const double *__restrict__ u,
                                                 double *__restrict__ part) {
  __shared__ double red[4];
  double s = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)LZ_T + threadIdx.x; i < n; i += (int64_t)gridDim.x * LZ_T)
    s += v[i] * u[i];
  const double t = lz_block_sum(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// w = M~^-1 u - alpha v_j - beta_{j-1} v_{j-1} (alpha from the partials, kept in
// alpha_out) and the partial sums of v_i.M~ w for i = i0 .. i0 + LZ_G - 1 <= j;
// write = false: w is there already
constexpr int LZ_G = 8;
__global__ __launch_bounds__(LZ_T) void k_lz_step(LzArgs a, int j, int i0, bool write,
                                                  const double *__restrict__ Vb, int64_t ldv,
                                                  const double *__restrict__ u,
                                                  const double *__restrict__ apart,
                                                  const double *__restrict__ beta,
                                                  double *__restrict__ alpha_out, double *w,
                                                  double *__restrict__ part) {
  __shared__ double red[4];
  const double al = write ? lz_total(apart, red) : 0.0;
  if (write && blockIdx.x == 0 && threadIdx.x == 0) *alpha_out = al;
  const double be = write && j > 0 ? *beta : 0.0;
  const double *v = Vb + j * ldv, *vp = j > 0 ? v - ldv : v;
  const int ng = min(LZ_G, j + 1 - i0);
  double s[LZ_G];
#pragma unroll
  for (int g = 0; g < LZ_G; ++g) s[g] = 0.0;
  lz_rows(a, [&](int64_t i) {
    double wi;
    if (write) {
      wi = a.minv[i] * u[i] - al * v[i] - be * vp[i];
      w[i] = wi;
    } else {
      wi = w[i];
    }
    const double mw = a.m[i] * wi;
#pragma unroll
    for (int g = 0; g < LZ_G; ++g)
      if (g < ng) s[g] += Vb[(i0 + g) * ldv + i] * mw;
  });
  lz_atoms(a, [&](int I, int k) {
    const int64_t r = a.nn + (int64_t)I * a.nf + k;
    const bool on = k < a.nf;
    double wi = 0.0;
    if (write) {
      const double uk = on ? u[r] : 0.0;
      for (int l = 0; l < a.nf; ++l) {
        const double ul = __shfl(uk, l, 16);
        if (on) wi += a.inv[((int64_t)I * a.nf + k) * a.nf + l] * ul;
      }
      if (on) {
        wi = wi - al * v[r] - be * vp[r];
        w[r] = wi;
      }
    } else if (on) {
      wi = w[r];
    }
    const double mw = lz_block_row(a, I, k, wi);
#pragma unroll
    for (int g = 0; g < LZ_G; ++g)
      if (g < ng && on) s[g] += Vb[(i0 + g) * ldv + r] * mw;
  });
#pragma unroll
  for (int g = 0; g < LZ_G; ++g) {
    if (g >= ng) break;
    const double t = lz_block_sum(s[g], red);
    if (threadIdx.x == 0) part[(int64_t)(i0 + g) * LZ_NP + blockIdx.x] = t;
  }
}

// w -= sum_{i <= j} c_i v_i (classical Gram-Schmidt against the Lanczos basis)
// with c_i from the partials; partial sums of w.M~ w
constexpr int LZ_MAXC = 1000;
__global__ __launch_bounds__(LZ_T) void k_lz_reorth(LzArgs a, int j, const double *__restrict__ Vb,
                                                    int64_t ldv, const double *__restrict__ cpart,
                                                    double *w, double *__restrict__ part) {
  __shared__ double red[4], c[LZ_MAXC];
  // one wave per coefficient
  for (int i = threadIdx.x / 64; i <= j; i += LZ_T / 64) {
    double s = 0.0;
    for (int q = threadIdx.x % 64; q < LZ_NP; q += 64) s += cpart[(int64_t)i * LZ_NP + q];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (threadIdx.x % 64 == 0) c[i] = s;
  }
  __syncthreads();
  double s = 0.0;
  lz_rows(a, [&](int64_t r) {
    double acc = 0.0;
#pragma unroll 4
    for (int i = 0; i <= j; ++i) acc += c[i] * Vb[i * ldv + r];
    const double wr = w[r] - acc;
    w[r] = wr;
    s += a.m[r] * wr * wr;
  });
  lz_atoms(a, [&](int I, int k) {
    const int64_t r = a.nn + (int64_t)I * a.nf + k;
    double wr = 0.0;
    if (k < a.nf) {
      double acc = 0.0;
#pragma unroll 4
      for (int i = 0; i <= j; ++i) acc += c[i] * Vb[i * ldv + r];
      wr = w[r] - acc;
      w[r] = wr;
    }
    s += wr * lz_block_row(a, I, k, wr);
  });
  const double t = lz_block_sum(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// theta_max of the k x k tridiagonal (alpha, beta), plus |beta_k|: the smallest
// double with every eigenvalue below it by Sturm counts, 64 probes at a time
// (one wave; one probe at a time took 95 us)
__global__ __launch_bounds__(64) void k_tridiag_bound(int k, const double *__restrict__ alpha,
                                                      const double *__restrict__ beta,
                                                      double *__restrict__ out) {
  double lo = 1e300, hi = -1e300;
  for (int i = 0; i < k; ++i) {
    double r = (i > 0 ? fabs(beta[i - 1]) : 0.0) + (i < k - 1 ? fabs(beta[i]) : 0.0);
    lo = fmin(lo, alpha[i] - r);
    hi = fmax(hi, alpha[i] + r);
  }
  for (int it = 0; it < 200; ++it) {
    const double mid = 0.5 * (lo + hi);
    if (!(mid > lo && mid < hi)) break;
    // lane l probes lo + (l + 1)/65 (hi - lo), clamped between the ends
    const double x = fmin(fmax(lo + (hi - lo) * ((threadIdx.x + 1) / 65.0), lo), hi);
    int cnt = 0;
    double d = 1.0;
    for (int i = 0; i < k; ++i) {
      const double b2 = i > 0 ? beta[i - 1] * beta[i - 1] : 0.0;
      d = alpha[i] - x - (i > 0 ? b2 / d : 0.0);
      if (d == 0.0) d = -1e-300;
      if (d < 0.0) ++cnt;
    }
    // lanes whose probe has every eigenvalue below it
    const uint64_t above = __ballot(cnt >= k);
    const int first = above ? __ffsll((unsigned long long)above) - 1 : 64;
    const double nhi = first < 64 ? __shfl(x, first) : hi, nlo = first > 0 ? __shfl(x, first - 1) : lo;
    if (nhi == hi && nlo == lo) {   // the probes fell on the ends: halve
      double dm = 1.0;
      int c = 0;
      for (int i = 0; i < k; ++i) {
        const double b2 = i > 0 ? beta[i - 1] * beta[i - 1] : 0.0;
        dm = alpha[i] - mid - (i > 0 ? b2 / dm : 0.0);
        if (dm == 0.0) dm = -1e-300;
        if (dm < 0.0) ++c;
      }
      if (c >= k) hi = mid;
      else lo = mid;
      continue;
    }
    hi = nhi;
    lo = nlo;
  }
  if (threadIdx.x == 0) out[0] = hi + fabs(beta[k - 1]);
}

extern "C" efe_status efe_spectrum_upper_bound(efe_ctx *c, const double *v0, int32_t steps,
                                               double *b_out) {
  if (!c) return EFE_EINVAL;
  if (!v0 || !b_out || steps < 1 || steps > 1000) EFE_FAIL(c, EFE_EINVAL, "bad arguments");
  if (!c->have_potential) EFE_FAIL(c, EFE_ESTATE, "no potential set");
  efe_status s;
  const int64_t rows = c->rows, nn = c->n_nodes, ne = c->n_enr;
  double *buf, *sc;
  // the Lanczos basis V_0 .. V_{steps-1}, then u (= H v), w, x (= M~^-1 u)
  if ((s = efe_ws(c, 20, (size_t)rows * (steps + 3) * 8, (void **)&buf))) return s;
  const size_t npart = (size_t)(steps + 2) * LZ_NP, nsc = 2 * (size_t)steps + 8 + npart;
  if ((s = efe_ws(c, 21, nsc * 8, (void **)&sc))) return s;
  double *Vb = buf, *u = buf + (int64_t)steps * rows, *w = u + rows, *x = w + rows;
  double *alpha = sc, *beta = sc + steps, *res = sc + 2 * steps;
  double *part = sc + 2 * steps + 8;                 // one row: v.u, or norms
  double *cpart = part + 2 * LZ_NP;                  // a row per basis vector
  HIPCHK(c, hipMemsetAsync(sc, 0, nsc * 8, c->stream));
  const int nbe = ne ? (int)std::min<int64_t>(cdiv(c->natoms, LZ_T / 16), LZ_NP / 8) : 0;
  const int nbc = (int)std::min<int64_t>(cdiv(nn, LZ_T), LZ_NP - LZ_NP / 8), nb = nbc + nbe;
  const LzArgs a{nn,      ne,         ne ? c->natoms : 0, c->nf, nbc, c->d_m_int,
                 c->d_minv, c->d_Mee, c->d_Mee_inv};
  double *npart_ = part + LZ_NP;
  k_lz_start<<<nb, LZ_T, 0, c->stream>>>(a, v0, u, npart_);
  k_lz_scale<<<nb, LZ_T, 0, c->stream>>>(rows, npart_, u, Vb, nullptr);
  for (int j = 0; j < steps; ++j) {
    double *v = Vb + (int64_t)j * rows;
    if ((s = efe_apply_H_internal(c, v, 1, false, v + nn, 1, u, 1, 1, EFE_FP64))) return s;
    // alpha_j = v^T H v; w = M~^-1 H v - alpha v - beta v_prev and its products
    // with the basis, once more against the whole basis, its norm
    k_lz_dot<<<nb, LZ_T, 0, c->stream>>>(rows, v, u, part);
    for (int i0 = 0; i0 <= j; i0 += LZ_G)
      k_lz_step<<<nb, LZ_T, 0, c->stream>>>(a, j, i0, i0 == 0, Vb, rows, u, part,
                                           j > 0 ? &beta[j - 1] : nullptr, &alpha[j], w, cpart);
    k_lz_reorth<<<nb, LZ_T, 0, c->stream>>>(a, j, Vb, rows, cpart, w, npart_);
    // v_{j+1} = w / beta_j (the last one is not kept)
    double *vn = j + 1 < steps ? Vb + (int64_t)(j + 1) * rows : x;
    k_lz_scale<<<nb, LZ_T, 0, c->stream>>>(rows, npart_, w, vn, &beta[j]);
  }
  k_tridiag_bound<<<1, 64, 0, c->stream>>>(steps, alpha, beta, res);
  HIPCHK(c, hipGetLastError());
  HIPCHK(c, hipMemcpyAsync(b_out, res, 8, hipMemcpyDeviceToHost, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return EFE_OK;
}
