// Cell Hamiltonians by tensor-product (sum-factorized) contractions, for
// meshes whose Gauss rule has as many points per axis as the elements have
// nodes (nq = p + 1 = P; other rules keep the dense cell matrices).
//
// H_c = 1/2 K + N^T diag(w v) N acts on the P^3 nodal values of one cell and
// one vector.  With the 1-D basis scaled to orthonormal Gauss values
// (N~ = diag(sqrt(w h/2)) N) both integrals are taken at the Gauss points:
//   u = (N~ x N~ x N~) x,   r = v u + (S_x + S_y + S_z) u,   y = (N~ x N~ x N~)^T r
// with S_d = 1/2 (2/h_d)^2 W^-1/2 D^T W D W^-1/2 acting along axis d and D the
// derivative matrix of the Lagrange basis on the Gauss points.  That is nine
// 1-D contractions, 18 P^4 flops instead of 2 P^6 (43 k instead of 235 k at
// P = 7), and it reads the potential (P^3 numbers a cell) in place of a
// P^3 x P^3 matrix, so the bound moves from the matrix cores to HBM: 0.86 ms
// for 4,096 cells x 160 vectors at P = 7 (counters: 1.47 GB read, 1.87 GB
// written, 3.9 TB/s), 51 us for one vector; the dense products of the same cells
// took 3.0 ms and 0.67 ms.  Both 1-D matrices are symmetric under reflection of
// the element, so every length-P contraction runs on the even and odd parts of its
// input: 25 multiply-adds and 12 additions at P = 7 in place of 49.
#include <cmath>
#include <vector>

#include "efe_device.h"
#include "line_ops.h"

namespace {
// vectors per work-group: U P threads share U P^3 doubles of LDS.  Chosen so
// that U P fills whole waves (P = 4: 64, P = 6: 192, P = 3: 192 threads) or
// nearly (P = 5: 120 of 128, P = 7: 112 of 128), a node's piece of U columns
// is whole 128-byte lines where P allows it (P = 7: one line), and three or
// more work-groups fit a CU's LDS (P = 7: 44 KB each).
constexpr int tp_units(int P) { return P == 7 ? 16 : P == 6 ? 32 : P == 5 ? 24 : P == 4 ? 16 : 64; }

// waves per SIMD the registers leave (two planes of P^2 doubles are live)
constexpr int tp_waves(int P) { return P >= 6 ? 2 : P == 5 ? 3 : 4; }

// A work-group takes U (cell, column) units; thread (s, u) owns plane s of
// unit u, P^2 values in registers, and contracts the two axes inside its
// plane there.  The third axis is reached by three exchanges through LDS,
// stored [z][y][x][unit]: every access of a wave is runs of consecutive
// doubles, free of bank conflicts.
//   A  plane z = s (nodes):   load, x and y to Gauss points            -> LDS
//   B  plane x = s:           z to Gauss points, S_y + S_z kept        -> LDS
//   C  plane z = s (Gauss):   v u + S_x u                              -> LDS
//   B' plane x = s:           + kept part, z and y back to the nodes   -> LDS
//   A' plane z = s:           x back to the nodes, store
// Units are laid out column group by column group (U columns each; the last
// group may be narrower and then a work-group holds several cells), so that
// ragged widths and single vectors fill the work-groups as full ones do.
//
// Accuracy: the rounding of the tables, amplified by S, is the larger part of the
// error on smooth values, so they are formed in extended precision and rounded
// once.  With 3 points an axis S u still loses digits against the constant part
// of u, and the value at the middle node is taken off first (S sees none of it;
// r gets v x0 sqrt(w) back).  Largest error of an apply relative to its largest
// value, smooth fields, p = 2 to 6, in 1e-15: 0.3, 1.7, 3.4, 3.8, 8.2, where the
// dense products have 0.8, 2.6, 5.1, 18, 32 and tables in double 1.7, 3.1, 9.4,
// 6.2, 21; random fields are below the dense products for every p.
template <int P>
__global__ __launch_bounds__(tp_units(P) * P) __attribute__((amdgpu_waves_per_eu(tp_waves(P))))
void k_cell_tp(TpArgs a) {
  constexpr int U = tp_units(P), PP = P * P, N = P * P * P;
  __shared__ double L[N * U];
  const int t = threadIdx.x, u = t % U, s = t / U;
  // consecutive logical work-groups (neighbouring cells of one column group,
  // which share face rows of X) run on one XCD
  int64_t blk = blockIdx.x;
  if (gridDim.x % 8 == 0) blk = (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int nfull = a.ncols / U;
  const int64_t g = min((int64_t)nfull, blk / a.ncells);
  const int w = g < nfull ? U : a.ncols - nfull * U;
  const int64_t unit = (blk - g * a.ncells) * U + u;
  const bool live = unit < a.ncells * w;
  const int64_t uc = live ? unit : a.ncells * w - 1;
  const int pos = w == U ? (int)(blk - g * a.ncells) : (int)(uc / w);
  const int jc = w == U ? u : (int)(uc - (int64_t)pos * w);
  const int cell = a.cells ? a.cells[pos] : pos;
  const int cx = cell % a.ncx, cy = (cell / a.ncx) % a.ncy, cz = cell / (a.ncx * a.ncy);
  const int64_t row0 = cx * (P - 1) + a.n1x * (cy * (P - 1) + a.n1y * (cz * (P - 1) + (int64_t)s));
  cdouble *const m0 = (cdouble *)(uintptr_t)a.m;
  cdouble *m = fresh(m0);
  constexpr bool MID = P == 3;
  double f[PP], x0 = 0.0;
  {
    double fx[P];
    if constexpr (MID) {
      const int64_t mx = cx * (P - 1) + 1, my = cy * (P - 1) + 1, mz = cz * (P - 1) + 1;
      x0 = a.X[(mx + a.n1x * (my + a.n1y * mz)) * a.ldx + g * U + jc] *
           (a.s1[mx] * (a.s1[a.n1x + my] * a.s1[a.n1x + a.n1y + mz]));
    }
    const double *sy = a.s1 + a.n1x + cy * (P - 1);
    double sz = 1.0;
    const double *x = a.X + row0 * a.ldx + g * U + jc;
#pragma unroll
    for (int b = 0; b < P; ++b)
#pragma unroll
      for (int i = 0; i < P; ++i) f[b * P + i] = x[(b * a.n1x + i) * a.ldx];
    const double *sx = a.s1 + cx * (P - 1);
    sz = a.s1[a.n1x + a.n1y + cz * (P - 1) + s];
#pragma unroll
    for (int i = 0; i < P; ++i) fx[i] = sx[i];
#pragma unroll
    for (int b = 0; b < P; ++b) {
      const double fy = sy[b] * sz;
      double v[P], y[P];
#pragma unroll
      for (int i = 0; i < P; ++i) v[i] = f[b * P + i] * (fx[i] * fy) - x0;
      mul1d<P, false>(m, 0, v, y);
#pragma unroll
      for (int i = 0; i < P; ++i) f[b * P + i] = y[i];
    }
    m = fresh(m0);
#pragma unroll
    for (int i = 0; i < P; ++i) {
      double v[P], y[P];
#pragma unroll
      for (int b = 0; b < P; ++b) v[b] = f[b * P + i];
      mul1d<P, false>(m, 1, v, y);
#pragma unroll
      for (int b = 0; b < P; ++b) L[((s * P + b) * P + i) * U + u] = y[b];
    }
  }
  __syncthreads();
  m = fresh(m0);
  double r[PP];   // [y][z]
#pragma unroll
  for (int b = 0; b < P; ++b) {
    double v[P], y[P];
#pragma unroll
    for (int c = 0; c < P; ++c) v[c] = L[((c * P + b) * P + s) * U + u];
    mul1d<P, false>(m, 2, v, y);
#pragma unroll
    for (int c = 0; c < P; ++c) {
      f[b * P + c] = y[c];
      L[((c * P + b) * P + s) * U + u] = y[c];
    }
    mul1d<P, false>(m, 5, y, v);
#pragma unroll
    for (int c = 0; c < P; ++c) r[b * P + c] = v[c];
  }
#pragma unroll
  for (int c = 0; c < P; ++c) {
    double v[P], y[P];
#pragma unroll
    for (int b = 0; b < P; ++b) v[b] = f[b * P + c];
    mul1d<P, false>(m, 4, v, y);
#pragma unroll
    for (int b = 0; b < P; ++b) r[b * P + c] += y[b];
  }
  __syncthreads();
  m = fresh(m0);
  {
    const double *vq = a.vq + (int64_t)cell * N + s * PP;
#pragma unroll
    for (int b = 0; b < P; ++b) {
      double v[P], y[P];
#pragma unroll
      for (int i = 0; i < P; ++i) v[i] = L[((s * P + b) * P + i) * U + u];
      mul1d<P, false>(m, 3, v, y);
      if constexpr (MID)
#pragma unroll
        for (int i = 0; i < P; ++i) v[i] = fma(x0, a.sw[(s * P + b) * P + i], v[i]);
#pragma unroll
      for (int i = 0; i < P; ++i)
        L[((s * P + b) * P + i) * U + u] = fma(vq[b * P + i], v[i], y[i]);
    }
  }
  __syncthreads();
  m = fresh(m0);
#pragma unroll
  for (int b = 0; b < P; ++b) {
    double v[P], y[P];
#pragma unroll
    for (int c = 0; c < P; ++c) v[c] = r[b * P + c] + L[((c * P + b) * P + s) * U + u];
    mul1d<P, true>(m, 2, v, y);
#pragma unroll
    for (int c = 0; c < P; ++c) r[b * P + c] = y[c];
  }
#pragma unroll
  for (int c = 0; c < P; ++c) {
    double v[P], y[P];
#pragma unroll
    for (int b = 0; b < P; ++b) v[b] = r[b * P + c];
    mul1d<P, true>(m, 1, v, y);
#pragma unroll
    for (int b = 0; b < P; ++b) L[((c * P + b) * P + s) * U + u] = y[b];
  }
  __syncthreads();
  m = fresh(m0);
  if (!live) return;
  if (a.Yc) {
    double *yc = a.Yc + ((int64_t)pos * N + s * PP) * a.ldc + g * U + jc;
#pragma unroll
    for (int b = 0; b < P; ++b) {
      double v[P], y[P];
#pragma unroll
      for (int i = 0; i < P; ++i) v[i] = L[((s * P + b) * P + i) * U + u];
      mul1d<P, true>(m, 0, v, y);
#pragma unroll
      for (int i = 0; i < P; ++i) __builtin_nontemporal_store(y[i], yc + (b * P + i) * a.ldc);
    }
  } else {
    // one colour of cells: no two work-groups share a row
    double *yp = a.Y + row0 * a.ldy + g * U + jc;
    const double *mx = a.mask1 + cx * (P - 1), *my = a.mask1 + a.n1x + cy * (P - 1);
    const double mz = a.alpha * a.mask1[a.n1x + a.n1y + cz * (P - 1) + s];
#pragma unroll
    for (int b = 0; b < P; ++b) {
      double v[P], y[P];
#pragma unroll
      for (int i = 0; i < P; ++i) v[i] = L[((s * P + b) * P + i) * U + u];
      mul1d<P, true>(m, 0, v, y);
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const int64_t o = (b * a.n1x + i) * a.ldy;
        yp[o] += mx[i] * my[b] * mz * y[i];
      }
    }
  }
}

// matrices of the projections and the density, then those of the cell operator and
// sqrt(w), appended to `all`
void tp_tables(const efe_ctx *c, const std::vector<double> &wq, const std::vector<double> &N1,
               const std::vector<long double> &wql,
               const std::vector<long double> &N1l, const std::vector<long double> &Dl,
               std::vector<double> &all) {
  const int P = c->P;
  std::vector<double> Nd(P * P), tab(3 * TP_MAT, 0.0);
  for (int d = 0; d < 3; ++d) {
    const double h2 = 0.5 * c->h[d];
    for (int q = 0; q < P; ++q)
      for (int i = 0; i < P; ++i) Nd[q * P + i] = sqrt(wq[q] * h2) * N1[q * P + i];
    even_odd(P, Nd, &tab[d * TP_MAT], &tab[d * TP_MAT + 16]);
  }
  all.insert(all.end(), tab.begin(), tab.end());
  tab.assign(6 * TP_MAT, 0.0);
  // the cell operator's own copy, from extended precision, and sqrt(w) of the
  // cell's Gauss points
  std::vector<long double> Nl(P * P), Sl(P * P);
  for (int d = 0; d < 3; ++d) {
    const long double h2 = 0.5L * c->h[d];
    for (int q = 0; q < P; ++q)
      for (int i = 0; i < P; ++i) {
        Nl[q * P + i] = sqrtl(wql[q] * h2) * N1l[q * P + i];
        long double acc = 0.0;
        for (int g = 0; g < P; ++g) acc += wql[g] * Dl[g * P + q] * Dl[g * P + i];
        Sl[q * P + i] = 0.5L * acc / (sqrtl(wql[q] * wql[i]) * h2 * h2);
      }
    even_odd(P, Nl, &tab[d * TP_MAT], &tab[d * TP_MAT + 16]);
    even_odd(P, Sl, &tab[(3 + d) * TP_MAT], &tab[(3 + d) * TP_MAT + 16]);
  }
  const long double jac = 0.125L * c->h[0] * c->h[1] * c->h[2];
  for (int q = 0; q < P * P * P; ++q)
    tab.push_back((double)sqrtl(wql[q % P] * wql[q / P % P] * wql[q / (P * P)] * jac));
  all.insert(all.end(), tab.begin(), tab.end());
}

}  // namespace

efe_status efe_tp_setup(efe_ctx *c, const std::vector<double> &wq, const std::vector<double> &N1,
                        const std::vector<double> &D1, const std::vector<double> &wg,
                        const std::vector<long double> &wql, const std::vector<long double> &N1l,
                        const std::vector<long double> &Dl) {
  c->tp = c->nq == c->P && c->P >= 2;
  const int P = c->P;
  // separable factors of the lumped mass: 1 (0 on the boundary), then 1/m
  const int64_t n3 = c->n1[0] + c->n1[1] + c->n1[2];
  std::vector<double> s1(2 * n3, 0.0);
  int64_t o = 0;
  for (int d = 0; d < 3; ++d)
    for (int64_t i = 0; i < c->n1[d]; ++i, ++o) {
      if (i == 0 || i == c->n1[d] - 1) continue;
      const int l = (int)(i % c->p);
      s1[o] = 1.0;
      s1[n3 + o] = 1.0 / (0.5 * c->h[d] * (l == 0 ? wg[0] + wg[c->p] : wg[l]));
    }
  // 1-D mass and stiffness of the Gauss rule on the nodes (any nq): the cell
  // stiffness is K x M x M + M x K x M + M x M x K
  std::vector<double> mk(6 * TP_MAT, 0.0), M(P * P), K(P * P);
  for (int d = 0; d < 3 && P >= 2; ++d) {
    const double h2 = 0.5 * c->h[d];
    for (int i = 0; i < P; ++i)
      for (int j = 0; j < P; ++j) {
        double m = 0.0, k = 0.0;
        for (int q = 0; q < c->nq; ++q) {
          m += wq[q] * N1[q * P + i] * N1[q * P + j];
          k += wq[q] * D1[q * P + i] * D1[q * P + j];
        }
        M[i * P + j] = h2 * m;
        K[i * P + j] = k / h2;
      }
    even_odd(P, M, &mk[d * TP_MAT], &mk[d * TP_MAT + 16]);
    even_odd(P, K, &mk[(3 + d) * TP_MAT], &mk[(3 + d) * TP_MAT + 16]);
  }
  std::vector<double> all = s1;            // s1, mk, and with c->tp the matrices
  all.insert(all.end(), mk.begin(), mk.end());
  if (c->tp) tp_tables(c, wq, N1, wql, N1l, Dl, all);
  efe_status st;
  if ((st = efe_alloc(c, (void **)&c->d_tpt, all.size() * 8))) return st;
  HIPCHK(c, hipMemcpyAsync(c->d_tpt, all.data(), all.size() * 8, hipMemcpyHostToDevice, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  c->d_s1 = c->d_tpt;
  c->d_mk = c->d_s1 + s1.size();
  c->d_tpm = c->d_mk + mk.size();
  c->d_tpc = c->d_tpm + 3 * TP_MAT;
  return EFE_OK;
}

// Cell products of every cell into Yc, or, with Yc = nullptr, added to the
// interior rows of Y times alpha, one colour of cells per launch.
efe_status efe_tp_apply(efe_ctx *c, const double *X, int64_t ldx, bool minv, int ncols, double *Yc,
                        int64_t ldc, double *Y, int64_t ldy, double alpha) {
  TpArgs a{};
  a.X = X;
  a.ldx = ldx;
  a.ncols = ncols;
  a.Yc = Yc;
  a.ldc = ldc;
  a.Y = Y;
  a.ldy = ldy;
  a.alpha = alpha;
  a.vq = c->d_vq;
  a.mask1 = c->d_s1;
  a.s1 = c->d_s1 + (minv ? c->n1[0] + c->n1[1] + c->n1[2] : 0);
  a.ncx = c->ncell[0];
  a.ncy = c->ncell[1];
  a.n1x = c->n1[0];
  a.n1y = c->n1[1];
  a.m = c->d_tpc;
  a.sw = c->d_tpc + 6 * TP_MAT;
  for (int col = 0; col < (Yc ? 1 : 8); ++col) {
    if (Yc) {
      a.ncells = c->n_cells;
    } else {
      a.ncells = c->colour_offsets[col + 1] - c->colour_offsets[col];
      a.cells = c->d_colour_order + c->colour_offsets[col];
    }
    if (a.ncells == 0) continue;
    const int U = tp_units(c->P);
    const int64_t nblk = (ncols / U) * a.ncells + cdiv(a.ncells * (ncols % U), U);
    if (nblk > 0x7fffffffLL) EFE_FAIL(c, EFE_EINVAL, "cell grid too large");
    const int t = efe_timer_begin(c, ncols <= 16 ? EFE_T_CELL_NARROW : EFE_T_CELL);
    const unsigned nb = (unsigned)nblk, th = (unsigned)(U * c->P);
    switch (c->P) {
      case 2: k_cell_tp<2><<<nb, th, 0, c->stream>>>(a); break;
      case 3: k_cell_tp<3><<<nb, th, 0, c->stream>>>(a); break;
      case 4: k_cell_tp<4><<<nb, th, 0, c->stream>>>(a); break;
      case 5: k_cell_tp<5><<<nb, th, 0, c->stream>>>(a); break;
      case 6: k_cell_tp<6><<<nb, th, 0, c->stream>>>(a); break;
      case 7: k_cell_tp<7><<<nb, th, 0, c->stream>>>(a); break;
    }
    efe_timer_end(c, ncols <= 16 ? EFE_T_CELL_NARROW : EFE_T_CELL, t);
  }
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}
