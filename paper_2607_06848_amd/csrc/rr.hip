// Rayleigh-Ritz in FP64 (Eq. projectedKSEig) with the exact overlap M^E
// (Sec. III.B: the approximate inverse is used only inside the filter).
//
//   W  = H V                      (column chunks of 160)        
//   S  = V^T M V  (lumped mass on CFE rows, M^ee on enrichment rows)
//   Hp = V^T W
//   S = L L^T, A = L^-1 Hp L^-T, A = Q Lambda Q^T (block Jacobi), R = L^-T Q:
//   Hp R = S R Lambda, R^T S R = I, ascending Lambda
//   V <- V R, W <- W R (row blocks, in place),
//   resnorm_j = ||W e_j - lambda_j M V e_j||
// Every product runs on the FP64 matrix cores (dense.hip).
#include <algorithm>
#include <cmath>

#include "efe_device.h"

__global__ void k_resnorm(int64_t n_nodes, int64_t rows, int N, const double *__restrict__ W,
                          const double *__restrict__ V, int64_t ldv,
                          const double *__restrict__ m_int,
                          const double *__restrict__ MVE, const double *__restrict__ lam,
                          double *__restrict__ out) {
  __shared__ double red[4][64];
  const int j = blockIdx.y * 64 + threadIdx.x;
  double acc = 0.0;
  if (j < N) {
    for (int64_t r = blockIdx.x * 4 + threadIdx.y; r < rows; r += (int64_t)gridDim.x * 4) {
      const double mv = r < n_nodes ? m_int[r] * V[r * ldv + j] : MVE[(r - n_nodes) * N + j];
      const double w = (r < n_nodes && m_int[r] == 0.0) ? 0.0 : W[r * N + j];
      const double d = w - lam[j] * mv;
      acc += d * d;
    }
  }
  red[threadIdx.y][threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.y == 0 && j < N)
    atomicAdd(&out[j], red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] +
                           red[3][threadIdx.x]);
}

__global__ void k_sqrt_inplace(int n, double *__restrict__ x) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = sqrt(x[i]);
}

// V[r0 + r][j] <- T[r][j] (boundary rows zero)
__global__ void k_copy_masked(int64_t r0, int64_t n_nodes, int64_t nr, int N,
                              const double *__restrict__ minv, const double *__restrict__ T,
                              double *__restrict__ V, int64_t ld) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= nr * N) return;
  const int64_t r = idx / N, g = r0 + r;
  const int j = idx % N;
  V[r * ld + j] = (g < n_nodes && minv[g] == 0.0) ? 0.0 : T[idx];
}

// ---- Blocks of up to 160 vectors.  Both Grams in one pass over the rows, and
// the rotation in place with the residual norms on the way: V and H V are read
// twice altogether and V is written once.
typedef double v4d_r __attribute__((ext_vector_type(4)));

// Partial sums of S = V^T M V (even work-groups) or Hp = V^T W (odd ones) over
// the rows of one pair of work-groups, as the 16 x 16 tiles on and above the
// diagonal, tile u of the list in wave u % 4.  16 rows at a time sit in LDS as V
// and M V (m V on CFE rows, M^ee V^E on enrichment rows) or W; the next 16 are
// on their way in registers.  Splitting the two Grams leaves 14 tiles a wave and
// two waves a SIMD to cover each other's operand reads; the second reading of V
// comes from the caches.  VEC: even leading dimensions, 16-byte aligned rows and
// an even N; the loads are unconditional, at clamped addresses, so that they stay
// in flight while the current rows are multiplied.  (128-wide tiles computed 49 k
// elements a row of the 160 x 160 upper triangle's 13 k: 3.9 ms for the pair at
// 0.91 M rows; both Grams in one work-group, 28 tiles a wave: 2.1 ms.)
struct GramArgs {
  int64_t nn, rows, ldv, ldw;
  int N, NB, ntile;
  const double *V, *W, *m, *MVE;
  double *part;
};

template <int UT, bool VEC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_gram_pair(GramArgs a) {
  constexpr int NC = 160;
  __shared__ __align__(16) double Xs[2][16][NC];
  const int t = threadIdx.x, wave = t / 64, lane = t % 64, li = lane % 16, lk = lane / 16;
  const bool hp = blockIdx.x & 1;
  const int64_t pair = blockIdx.x / 2, npair = gridDim.x / 2;
  const double *B = hp ? a.W : a.V;
  const int64_t ldb = hp ? a.ldw : a.ldv;
  const int np = 8 * a.NB;                  // column pairs of a staged row
  int ca[UT], cb[UT];                       // first columns of this wave's tiles
#pragma unroll
  for (int u = 0; u < UT; ++u) {
    int x = min(wave + 4 * u, a.ntile - 1), i = 0;
    while (x >= a.NB - i) {
      x -= a.NB - i;
      ++i;
    }
    ca[u] = __builtin_amdgcn_readfirstlane(16 * i);
    cb[u] = __builtin_amdgcn_readfirstlane(16 * (i + x));
  }
  v4d_r acc[UT];
#pragma unroll
  for (int u = 0; u < UT; ++u) acc[u] = (v4d_r){0.0, 0.0, 0.0, 0.0};
  // 16 rows x np pairs over 256 threads: five pairs a thread at 160 columns
  double2 v[5], w[5];
  double m[5];
  int rr[5], cc[5];
  bool in[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    const int idx = t + 256 * j;
    in[j] = idx < 16 * np;
    rr[j] = in[j] ? idx / np : 15;
    cc[j] = 2 * (idx % np);
  }
  auto load = [&](int64_t r0) {
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const int64_t row = min(r0 + rr[j], a.nn - 1);
      const double *vp = a.V + row * a.ldv, *wp = B + row * ldb;
      if constexpr (VEC) {
        const int c = min(cc[j], a.N - 2);
        v[j] = *(const double2 *)(vp + c);
        w[j] = *(const double2 *)(wp + c);
      } else {
        const int c = min(cc[j], a.N - 1), c1 = min(cc[j] + 1, a.N - 1);
        v[j] = make_double2(vp[c], vp[c1]);
        w[j] = make_double2(wp[c], wp[c1]);
      }
      m[j] = hp ? 1.0 : a.m[row];
    }
  };
  // columns past N and rows past the end count as zero
  auto store = [&](int64_t r0) {
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      if (!in[j]) continue;
      const bool on = r0 + rr[j] < a.nn, x0 = on && cc[j] < a.N, x1 = on && cc[j] + 1 < a.N;
      *(double2 *)&Xs[0][rr[j]][cc[j]] = make_double2(x0 ? v[j].x : 0.0, x1 ? v[j].y : 0.0);
      *(double2 *)&Xs[1][rr[j]][cc[j]] =
          make_double2(x0 ? m[j] * w[j].x : 0.0, x1 ? m[j] * w[j].y : 0.0);
    }
  };
  auto multiply = [&]() {
#pragma unroll 1
    for (int s = 0; s < 4; ++s) {
      const double *vs = &Xs[0][4 * s + lk][li], *ms = &Xs[1][4 * s + lk][li];
#pragma unroll
      for (int u = 0; u < UT; ++u)
        acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(vs[ca[u]], ms[cb[u]], acc[u], 0, 0, 0);
    }
  };
  const int64_t step = npair * 16;
  load(pair * 16);
  for (int64_t r0 = pair * 16; r0 < a.nn; r0 += step) {
    __syncthreads();
    store(r0);
    __syncthreads();
    load(r0 + step);
    multiply();
  }
  // enrichment rows, 16 at a time, by the first pairs
  for (int64_t r0 = a.nn + pair * 16; r0 < a.rows; r0 += step) {
    __syncthreads();
    for (int i = t; i < 16 * 16 * a.NB; i += 256) {
      const int r = i / (16 * a.NB), c = i % (16 * a.NB);
      const int64_t row = r0 + r;
      const bool on = row < a.rows && c < a.N;
      Xs[0][r][c] = on ? a.V[row * a.ldv + c] : 0.0;
      Xs[1][r][c] = !on ? 0.0 : hp ? a.W[row * a.ldw + c] : a.MVE[(row - a.nn) * a.N + c];
    }
    __syncthreads();
    multiply();
  }
  // accumulator v of lane l: row 4 v + l/16 of the tile, column l%16
  double *p = a.part + (int64_t)blockIdx.x * a.ntile * 256;
#pragma unroll
  for (int u = 0; u < UT; ++u) {
    const int tl = wave + 4 * u;
    if (tl >= a.ntile) break;
#pragma unroll
    for (int q = 0; q < 4; ++q) p[(int64_t)tl * 256 + 16 * (4 * q + lk) + li] = acc[u][q];
  }
}

// sums of the partial tiles in work-group order, into both triangles of S
// (blockIdx.y = 0) or Hp
__global__ __launch_bounds__(256) void k_gram_sum(int npair, int N, int NB, int ntile,
                                                  const double *__restrict__ part,
                                                  double *__restrict__ S,
                                                  double *__restrict__ Hp) {
  const int tl = blockIdx.x, e = threadIdx.x;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int g = 0; g < npair; g += 4)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (g + q < npair) s[q] += part[((2 * (int64_t)(g + q) + blockIdx.y) * ntile + tl) * 256 + e];
  const double x = (s[0] + s[1]) + (s[2] + s[3]);
  int y = tl, i = 0;
  while (y >= NB - i) {
    y -= NB - i;
    ++i;
  }
  const int r = 16 * i + e / 16, c = 16 * (i + y) + e % 16;
  double *C = blockIdx.y ? Hp : S;
  // inside a diagonal tile the upper triangle counts
  if (r < N && c < N && r <= c) {
    C[(int64_t)r * N + c] = x;
    C[(int64_t)c * N + r] = x;
  }
}

// X R for the rows of a block, boundary rows zero.  RES = false: written back to
// X in place (a work-group reads its 64 rows to the end before it writes them).
// RES = true (X = W): only the sums over the rows of (W R - lambda m V)^2 per
// column are kept, V the rotated block.  A wave holds 16 rows; R, padded to
// whole tiles with zeros, streams through LDS 16 rows at a time; a lane's four
// operand values of a chunk are adjacent in memory (rows 4 (l/16) + s of R meet
// them in step s).  VEC: even ld, 16-byte aligned rows and N % 4 == 0; every
// load is then unconditional and stays in flight during the products before
// its use (0.91 M rows x 160: 1.1 ms for V, 43 TFLOP/s, and 1.6 ms for the
// residuals; products into a buffer, masked copies and a residual pass took 5.5).
// Work-groups take 64 rows at a time; their sums go to
// res[work-group][N].
struct RotArgs {
  int64_t r0, r1, nn, ldx, ldv;
  int N;
  double *X;
  const double *V, *R, *m, *lam;
  double *res;
};

// R padded to 16 ceil(N/16) rows of nc columns
__global__ void k_pad_rot(int N, int nr, int nc, const double *__restrict__ R,
                          double *__restrict__ P) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nr * nc) return;
  const int r = i / nc, c = i % nc;
  P[i] = r < N && c < N ? R[(int64_t)r * N + c] : 0.0;
}

template <int CBM, bool RES, bool VEC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CBM < 6 ? 4 : 2)))
void k_rotate(RotArgs a) {
  constexpr int NC = 16 * CBM;
  __shared__ __align__(16) double Rs[2][16][NC];
  __shared__ double red[4][NC];
  const int t = threadIdx.x, wave = t / 64, lane = t % 64, li = lane % 16, lk = lane / 16;
  const int N = a.N, NCH = (N + 15) / 16;
  double rs[RES ? CBM : 1];
#pragma unroll
  for (int cb = 0; cb < (RES ? CBM : 1); ++cb) rs[cb] = 0.0;
  for (int64_t b0 = a.r0 + blockIdx.x * (int64_t)64; b0 < a.r1; b0 += (int64_t)gridDim.x * 64) {
    const double *xp = a.X + min(b0 + 16 * wave + li, a.r1 - 1) * a.ldx;
    v4d_r acc[CBM];
#pragma unroll
    for (int cb = 0; cb < CBM; ++cb) acc[cb] = (v4d_r){0.0, 0.0, 0.0, 0.0};
    double x[CBM];   // 16 x NC elements of R over 256 threads
    auto rload = [&](int ch) {
#pragma unroll
      for (int j = 0; j < CBM; ++j) x[j] = a.R[ch * 16 * NC + t + 256 * j];
    };
    auto rstore = [&](int buf) {
#pragma unroll
      for (int j = 0; j < CBM; ++j) (&Rs[buf][0][0])[t + 256 * j] = x[j];
    };
    auto aload = [&](int ch, double (&d)[4]) {
      // columns past N meet zero rows of R
      const int c = 16 * ch + 4 * lk;
      if constexpr (VEC) {
        const double *p = xp + min(c, N - 4);
        const double2 u0 = *(const double2 *)p, u1 = *(const double2 *)(p + 2);
        d[0] = u0.x;
        d[1] = u0.y;
        d[2] = u1.x;
        d[3] = u1.y;
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) d[s] = xp[min(c + s, N - 1)];
      }
    };
    double v0[4], v1[4];
    auto step = [&](int ch, const double (&v)[4], double (&vn)[4], int buf) {
      const bool more = ch + 1 < NCH;
      if (more) {
        rload(ch + 1);
        aload(ch + 1, vn);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int cb = 0; cb < CBM; ++cb)
          acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[s], Rs[buf][4 * lk + s][16 * cb + li],
                                                         acc[cb], 0, 0, 0);
      if (more) rstore(buf ^ 1);
      __syncthreads();
    };
    rload(0);
    aload(0, v0);
    rstore(0);
    __syncthreads();
    for (int ch = 0; ch < NCH; ch += 2) {
      step(ch, v0, v1, 0);
      if (ch + 1 < NCH) step(ch + 1, v1, v0, 1);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t r = b0 + 16 * wave + 4 * q + lk;
      if (r >= a.r1) continue;
      const double m = r < a.nn ? a.m[r] : 1.0;
#pragma unroll
      for (int cb = 0; cb < CBM; ++cb) {
        const int c = 16 * cb + li;
        if (c >= N) continue;
        const double y = m != 0.0 ? acc[cb][q] : 0.0;
        if constexpr (RES) {
          const double d = y - a.lam[c] * (m * a.V[r * a.ldv + c]);
          rs[cb] += d * d;
        } else {
          a.X[r * a.ldx + c] = y;
        }
      }
    }
  }
  if constexpr (RES) {
#pragma unroll
    for (int cb = 0; cb < CBM; ++cb) {
      double s = rs[cb];
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      if (lk == 0) red[wave][16 * cb + li] = s;
    }
    __syncthreads();
    if (t < N)
      a.res[(int64_t)blockIdx.x * N + t] = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
  }
}

// out[j] += sum over the work-groups of res[g][j], in order
__global__ __launch_bounds__(64) void k_res_sum(int nwg, int N, const double *__restrict__ res,
                                                double *__restrict__ out) {
  const int j = blockIdx.x;
  double s = 0.0;
  for (int g = threadIdx.x; g < nwg; g += 64) s += res[(int64_t)g * N + j];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (threadIdx.x == 0) out[j] += s;
}

constexpr int RR_WG = 256;      // pairs of work-groups of the Gram pass (one a CU)
constexpr int ROT_WG = 1024;

static efe_status gram_pair(efe_ctx *c, const GramArgs &a, double *S, double *Hp) {
  const int npair = (int)std::min<int64_t>(RR_WG, cdiv(a.rows, 16)), nwg = 2 * npair;
  const int ut = (int)cdiv(a.ntile, 4);
  const bool vec = a.ldv % 2 == 0 && a.ldw % 2 == 0 && (uintptr_t)a.V % 16 == 0 &&
                   (uintptr_t)a.W % 16 == 0 && a.N % 2 == 0;
#define GO(U)                                                      \
  do {                                                             \
    if (vec) k_gram_pair<U, true><<<nwg, 256, 0, c->stream>>>(a);  \
    else k_gram_pair<U, false><<<nwg, 256, 0, c->stream>>>(a);     \
  } while (0)
  if (ut <= 1) GO(1);
  else if (ut <= 3) GO(3);
  else if (ut <= 7) GO(7);
  else GO(14);
#undef GO
  k_gram_sum<<<dim3(a.ntile, 2), 256, 0, c->stream>>>(npair, a.N, a.NB, a.ntile, a.part, S, Hp);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}

// columns of the register tile of k_rotate
static int rot_tile(int N) { return N <= 16 ? 1 : N <= 48 ? 3 : N <= 96 ? 6 : 10; }

// rows r0 .. r1 of X (R padded to the tile); out: the residual sums are added there
static efe_status rotate(efe_ctx *c, const RotArgs &a, double *out) {
  if (a.r1 <= a.r0) return EFE_OK;
  const int nwg = (int)std::min<int64_t>(ROT_WG, cdiv(a.r1 - a.r0, 64));
  const bool vec = a.ldx % 2 == 0 && (uintptr_t)a.X % 16 == 0 && a.N % 4 == 0;
#define GO(B)                                                                    \
  do {                                                                           \
    if (out && vec) k_rotate<B, true, true><<<nwg, 256, 0, c->stream>>>(a);      \
    else if (out) k_rotate<B, true, false><<<nwg, 256, 0, c->stream>>>(a);       \
    else if (vec) k_rotate<B, false, true><<<nwg, 256, 0, c->stream>>>(a);       \
    else k_rotate<B, false, false><<<nwg, 256, 0, c->stream>>>(a);               \
  } while (0)
  switch (rot_tile(a.N)) {
    case 1: GO(1); break;
    case 3: GO(3); break;
    case 6: GO(6); break;
    default: GO(10);
  }
#undef GO
  if (out) k_res_sum<<<a.N, 64, 0, c->stream>>>(nwg, a.N, a.res, out);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}

// rows of the in-place rotation per pass
static int64_t rot_rows(int32_t N) { return std::max<int64_t>(64, (int64_t)(256 << 20) / (8 * N)); }

extern "C" efe_status efe_rayleigh_ritz(efe_ctx *c, double *V, int32_t N, int64_t ld,
                                        double *lambda, double *resnorm) {
  if (!c) return EFE_EINVAL;
  if (!V || !lambda || N < 1 || ld < N) EFE_FAIL(c, EFE_EINVAL, "bad arguments");
  if (!c->have_potential) EFE_FAIL(c, EFE_ESTATE, "no potential set");
  efe_status s;
  const int64_t rows = c->rows, nn = c->n_nodes, ne = c->n_enr;
  const int64_t rb = std::min<int64_t>(rows, rot_rows(N));
  const int64_t N2 = (int64_t)N * N;
  double *W, *T = nullptr, *MVE, *S, *Hp, *Li, *T1, *Qe, *R, *work;
  int *iwork, *flag;
  if ((s = efe_ws(c, 5, (size_t)rows * N * 8, (void **)&W))) return s;
  if ((s = efe_ws(c, 6, (size_t)std::max<int64_t>(ne, 1) * N * 8, (void **)&MVE))) return s;
  if ((s = efe_ws(c, 10, (size_t)6 * N2 * 8 + 256, (void **)&S))) return s;
  Hp = S + N2;
  Li = Hp + N2;
  T1 = Li + N2;
  Qe = T1 + N2;
  R = Qe + N2;
  flag = (int *)(R + N2);
  if ((s = efe_ws(c, 13, efe_syev_work(N) * 8, (void **)&work))) return s;
  if ((s = efe_ws(c, 14, efe_syev_iwork(N) * sizeof(int), (void **)&iwork))) return s;
  const bool one = N <= EFE_COL_CHUNK;   // one register tile holds the columns
  double *part = nullptr;
  const int NB = (int)cdiv(N, 16), ntile = NB * (NB + 1) / 2;
  if (one) {
    // partial tiles of the Grams, then partial sums and padded R of the rotation
    const size_t np = std::max((size_t)2 * RR_WG * ntile * 256, (size_t)ROT_WG * N + 16 * NB * 160);
    if ((s = efe_ws(c, 16, np * 8, (void **)&part))) return s;
  } else if ((s = efe_ws(c, 3, (size_t)rb * N * 8, (void **)&T))) {
    return s;
  }
  const int t_rr = efe_timer_begin(c, EFE_T_RR);
  // W = H V, chunk by chunk
  for (int32_t j0 = 0; j0 < N; j0 += EFE_COL_CHUNK) {
    const int32_t nc = std::min<int32_t>(EFE_COL_CHUNK, N - j0);
    if ((s = efe_apply_H_internal(c, V + j0, ld, false, V + nn * ld + j0, ld, W + j0, N, nc,
                                  EFE_FP64)))
      return s;
  }
  // S = V^T M V, Hp = V^T W (both are symmetric, H^E is: only the upper
  // triangle is formed): in one pass for blocks of one register tile, else as
  // tall-skinny products whose sum over rows is split across work-groups
  if (ne && (s = efe_dgemm(c, false, false, ne, N, ne, 1.0, c->d_Mee, ne, V + nn * ld, ld, 0.0, MVE,
                           N)))
    return s;
  if (one) {
    const GramArgs ga{nn, rows, ld, N, N, NB, ntile, V, W, c->d_m_int, MVE, part};
    if ((s = gram_pair(c, ga, S, Hp))) return s;
  } else {
    HIPCHK(c, hipMemsetAsync(S, 0, (size_t)2 * N2 * 8, c->stream));
    if ((s = efe_gram_sym(c, N, nn, V, ld, V, ld, S, N, c->d_m_int))) return s;
    if (ne && (s = efe_gram_sym(c, N, ne, V + nn * ld, ld, MVE, N, S, N))) return s;
    if ((s = efe_gram_sym(c, N, nn, V, ld, W, N, Hp, N))) return s;
    if (ne && (s = efe_gram_sym(c, N, ne, V + nn * ld, ld, W + nn * N, N, Hp, N))) return s;
    if ((s = efe_mirror_upper(c, N, S, N)) || (s = efe_mirror_upper(c, N, Hp, N))) return s;
  }
  // S = L L^T; Hp <- L^-1 Hp L^-T
  HIPCHK(c, hipMemsetAsync(flag, 0, sizeof(int), c->stream));
  if ((s = efe_potrf(c, N, S, N, flag))) return s;
  int hflag = 0;
  HIPCHK(c, hipMemcpyAsync(&hflag, flag, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  if (hflag) EFE_FAIL(c, EFE_ENUMERIC, "overlap of the block is not positive definite");
  if ((s = efe_trtri_lower(c, N, S, N, Li, N))) return s;
  if ((s = efe_dgemm(c, false, false, N, N, N, 1.0, Li, N, Hp, N, 0.0, T1, N))) return s;
  if ((s = efe_dgemm(c, false, true, N, N, N, 1.0, T1, N, Li, N, 0.0, Hp, N))) return s;
  // Hp = Q Lambda Q^T; R = L^-T Q
  if ((s = efe_syev_jacobi(c, N, Hp, N, lambda, Qe, work, iwork, &c->rr_sweeps))) return s;
  if ((s = efe_dgemm(c, true, false, N, N, N, 1.0, Li, N, Qe, N, 0.0, R, N))) return s;
  if (resnorm) HIPCHK(c, hipMemsetAsync(resnorm, 0, N * 8, c->stream));
  if (one) {
    // V <- V R in place; then the CFE rows' share of the residual norms from W
    // R, and W R on the enrichment rows, whose M^ee V R couples them
    const int nc = 16 * rot_tile(N), nr = 16 * NB;
    double *Rp = part + (size_t)ROT_WG * N;
    k_pad_rot<<<cdiv(nr * nc, 256), 256, 0, c->stream>>>(N, nr, nc, R, Rp);
    RotArgs ra{0, rows, nn, ld, ld, N, V, nullptr, Rp, c->d_m_int, lambda, part};
    if ((s = rotate(c, ra, nullptr))) return s;
    if (resnorm) {
      ra.X = W;
      ra.ldx = N;
      ra.V = V;
      ra.r1 = nn;
      if ((s = rotate(c, ra, resnorm))) return s;
      ra.r0 = nn;
      ra.r1 = rows;
      if ((s = rotate(c, ra, nullptr))) return s;
    }
  } else {
    // V <- V R, W <- W R, row block by row block through T
    for (int64_t r0 = 0; r0 < rows; r0 += rb) {
      const int64_t nr = std::min<int64_t>(rb, rows - r0);
      if ((s = efe_dgemm(c, false, false, nr, N, N, 1.0, V + r0 * ld, ld, R, N, 0.0, T, N))) return s;
      k_copy_masked<<<cdiv(nr * N, 256), 256, 0, c->stream>>>(r0, nn, nr, N, c->d_minv, T, V + r0 * ld,
                                                             ld);
      if (resnorm) {
        if ((s = efe_dgemm(c, false, false, nr, N, N, 1.0, W + r0 * N, N, R, N, 0.0, T, N))) return s;
        k_copy_masked<<<cdiv(nr * N, 256), 256, 0, c->stream>>>(r0, nn, nr, N, c->d_minv, T,
                                                               W + r0 * N, N);
      }
    }
  }
  if (resnorm) {
    if (ne && (s = efe_dgemm(c, false, false, ne, N, ne, 1.0, c->d_Mee, ne, V + nn * ld, ld, 0.0,
                             MVE, N)))
      return s;
    const int64_t r0 = one ? nn : 0;       // rows whose residual is still to sum
    if (rows > r0) {
      dim3 blkd(64, 4), grd((unsigned)std::min<int64_t>(cdiv(rows - r0, 4), 4096), cdiv(N, 64));
      k_resnorm<<<grd, blkd, 0, c->stream>>>(nn - r0, rows - r0, N, W + r0 * N, V + r0 * ld, ld,
                                            c->d_m_int, MVE, lambda, resnorm);
    }
    k_sqrt_inplace<<<cdiv(N, 256), 256, 0, c->stream>>>(N, resnorm);
  }
  efe_timer_end(c, EFE_T_RR, t_rr);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}
