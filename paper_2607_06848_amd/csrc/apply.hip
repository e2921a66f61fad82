// Application of the EFE Hamiltonian H^E = T^T Hhat T (Sec. II.B, Eq.
// Discrete_Eig_Gen_H), the exact overlap M^E and its approximate inverse
// (Eq. MEInvApprox) to a block of node-major vectors.
//
// T = [[I, -C^T], [0, I]] is applied when the operator is built: the coupling
// E = B - C H^cc of the orthogonalized basis to the nodes, the enrichment block
// H^phiphi - C B^T - E C^T and the projector rows P~^phi = P^phi - P^C C^T are
// formed in FP64 (setup.hip, couple.hip).  The apply of Y = alpha H^E X (+ the
// terms of the Chebyshev recurrence) then runs as
//   cells    Yc  = H_c s X^C_c                   (tensor products, every cell at once)
//   gather   Yp  = [E ; P^C] s X^C box by box    (MFMA)
//   sum      E s X^C, P^C s X^C and X^E atom by atom
//   dense    Y^E = alpha (E s X^C + H^E_ee X^E + P~^phi^T W) + ...,
//            W   = D (P^C s X^C + P~^phi X^E)    (MFMA)
//   nodes    Y^C = alpha (sum_c P_c^T Yc + E^T X^E + P^C^T W) + beta Z1 + gamma Z2
//                  + alpha G Cl                  (MFMA, one pass over the rows)
// in five launches (six where the columns leave a rest of 64-column parts, one more
// in FP32, whose gather takes E and P^C apart; one less without enrichment), with
// s = 1, or X = M~^-1 Z: s = 1/m and X^E = (M~^ee)^-1 Z^E formed by the sum step.
// Gauss rules with nq != p + 1 points, and BF16, add dense cell products H_c s
// X^C_c to Y^C in eight colour passes instead of the cells step (no two cells of a
// pass share a node); so do the tensor products without room for Yc.
#include <algorithm>

#include "efe_device.h"

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));

// Streams that a launch reads or writes once and that are far larger than the
// caches (the cells' products, the recurrence blocks, the coupling blocks, the
// partial rows) go with the non-temporal hint, so that they do not evict what
// is re-read through L2 (the rows of a box, the coefficient rows).  The hint changes
// cache policy only, not the values.
template <typename T>
__device__ inline T ld_nt(const T *p) {
  return __builtin_nontemporal_load(p);
}
template <typename T>
__device__ inline void st_nt(T v, T *p) {
  __builtin_nontemporal_store(v, p);
}
__device__ inline double2 ld_nt2(const double *p) {
  const v2d t = __builtin_nontemporal_load(reinterpret_cast<const v2d *>(p));
  return make_double2(t.x, t.y);
}
__device__ inline void st_nt2(double2 v, double *p) {
  const v2d t = {v.x, v.y};
  __builtin_nontemporal_store(t, reinterpret_cast<v2d *>(p));
}

// ------------------------------------------------------------------ pre
// One wave per group of 8 consecutive nodes, one lane per column (up to 192
// columns per pass, three per lane).  For every atom of the group's union
// the nine X^E rows are read once and applied to all eight nodes with the
// group-major coefficients (uniform over the wave, so they come through the
// scalar cache): Xh = X^C - C^T X^E, boundary rows 0.
constexpr int PRE_Q = 3;
__global__ __launch_bounds__(256) void k_pre(int64_t n_nodes, int ncols, const double *__restrict__ XC,
                                             int64_t ldx, const double *__restrict__ minv,
                                             const double *__restrict__ XE, int64_t lde,
                                             const int32_t *__restrict__ g_ptr,
                                             const int32_t *__restrict__ g_atom,
                                             const double *__restrict__ Cg, int nf,
                                             double *__restrict__ Xh, int64_t ldh) {
  const int64_t grp =
      (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
  const int lane = threadIdx.x % 64;
  const int64_t n0 = grp * 8;
  if (n0 >= n_nodes) return;
  const int nn = (int)min<int64_t>(8, n_nodes - n0);
  bool inner[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) inner[j] = j < nn && minv[n0 + j] != 0.0;
  const int32_t a0 = g_ptr[grp], a1 = g_ptr[grp + 1];
  for (int c0 = 0; c0 < ncols; c0 += 64 * PRE_Q) {
    double xh[PRE_Q][8];
#pragma unroll
    for (int q = 0; q < PRE_Q; ++q) {
      const int col = c0 + 64 * q + lane;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        // unconditional loads at clamped addresses keep every load of the
        // group in flight at once; the select drops what they brought in
        const double xv = XC[(n0 + min(j, nn - 1)) * ldx + min(col, ncols - 1)];
        xh[q][j] = (inner[j] && col < ncols) ? xv : 0.0;
      }
    }
    for (int32_t a = a0; a < a1; ++a) {
      const double *xe = XE + (int64_t)g_atom[a] * nf * lde;
      const double *cg = Cg + (int64_t)a * nf * 8;
      for (int k = 0; k < nf; ++k) {
        double v[PRE_Q];
#pragma unroll
        for (int q = 0; q < PRE_Q; ++q) {
          const int col = c0 + 64 * q + lane;
          v[q] = xe[(int64_t)k * lde + min(col, ncols - 1)];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const double cj = cg[k * 8 + j];
#pragma unroll
          for (int q = 0; q < PRE_Q; ++q) xh[q][j] -= cj * v[q];
        }
      }
    }
#pragma unroll
    for (int q = 0; q < PRE_Q; ++q) {
      const int col = c0 + 64 * q + lane;
      if (col >= ncols) continue;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (j >= nn) continue;
        Xh[(n0 + j) * ldh + col] = inner[j] ? xh[q][j] : 0.0;
      }
    }
  }
}

// ------------------------------------------------------------------ cell GEMM
// Matrix-core operations of the cell GEMM per element type: the operand
// fragments and accumulator layout of v_mfma_f64_16x16x4 (double) and
// v_mfma_f32_16x16x4 (float, FP32 accumulation), and the LDS row strides of
// the gathered block.
template <typename T>
struct CellMfma;
template <>
struct CellMfma<double> {
  typedef v4d acc_t;
  // LDS row stride for NC columns: the two 16-lane rows of a half-wave read
  // hit disjoint banks
  static constexpr int ncp(int NC) { return NC == 16 ? 16 : NC + 16; }
  __device__ static inline acc_t op(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // accumulator register v of lane l holds row 4 v + l/16
  __device__ static inline int row(int v, int lk) { return 4 * v + lk; }
};
typedef float v4f __attribute__((ext_vector_type(4)));
template <>
struct CellMfma<float> {
  typedef v4f acc_t;
  // LDS row stride for NC columns: the four 16-lane rows of a wave read hit
  // disjoint banks
  static constexpr int ncp(int NC) { return NC == 16 ? 16 : NC + 48; }
  __device__ static inline acc_t op(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // accumulator register v of lane l holds row 4 (l/16) + v
  __device__ static inline int row(int v, int lk) { return 4 * lk + v; }
};

template <typename T>
struct CellOps {
  int ncells, nparts;
  const int32_t *cells, *c2g;
  int nloc, RB, KS, ncols;
  const T *Ht;                     // cell Hamiltonian tiles
  const double *X;                 // CFE rows (even ld, 16-byte aligned)
  int64_t ldx;
  const double *scale, *minv;      // row scale of X (NULL: 1), 1/m (0 on the boundary)
  double *Y;                       // CFE rows, read-modify-write
  int64_t ldy;
  double alpha;
};

// waves per SIMD the wide tiles are compiled for: the FP64 accumulators of
// one row block x ten column blocks, or the FP32 ones of two, leave room for
// three; the FP32 ones of one row block for four
template <typename T, int RBW, int CBM>
constexpr int cell_waves() {
  return CBM == 1 ? 1 : (sizeof(T) == 8 || RBW > 1 ? 3 : 4);
}

// Dense cell GEMM of one colour pass, Y^C_c += alpha H_c (s X^C_c), for Gauss
// rules that the tensor-product form (cell_tp.hip) does not take (nq != p + 1).
// One work-group = one cell of the colour and a part of its row blocks, all
// (up to 160) columns.  Each wave keeps RBW row blocks x CBM column blocks of
// accumulators, so every matrix fragment loaded from memory feeds CBM MFMAs.
// The gathered rows stream through LDS in 16-row chunks, double buffered; the
// matrix fragments of the next chunk are loaded into registers while the
// current chunk is multiplied.  T = double (v_mfma_f64_16x16x4) or float
// (v_mfma_f32_16x16x4, FP32 accumulation).
template <typename T, int RBW, int CBM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(cell_waves<T, RBW, CBM>())))
void k_cell3(CellOps<T> a) {
  typedef CellMfma<T> M;
  typedef typename M::acc_t acc_t;
  constexpr int NC = CBM * 16, KC = 16;
  __shared__ T Xs[2][KC][M::ncp(NC)];
  __shared__ int32_t gs[16 * ((EFE_MAXLOC + 15) / 16)];
  __shared__ double gsc[16 * ((EFE_MAXLOC + 15) / 16)];
  const int b = blockIdx.x;
  const int xcd = b % 8, slot = b / 8;
  const int ci = (slot / a.nparts) * 8 + xcd;
  const int part = slot % a.nparts;
  if (ci >= a.ncells) return;
  const int cell = a.cells[ci];
  const int nloc = a.nloc, ncols = a.ncols;
  const int t = threadIdx.x, wave = t / 64, lane = t % 64, li = lane % 16, lk = lane / 16;
  const int NCH = (a.KS + 3) / 4;
  const int32_t *g = a.c2g + (int64_t)cell * nloc;
  for (int l = t; l < 16 * NCH; l += 256) {
    const int32_t node = g[min(l, nloc - 1)];
    gs[l] = node;
    gsc[l] = (l >= nloc || a.minv[node] == 0.0) ? 0.0 : (a.scale ? a.scale[node] : 1.0);
  }
  __syncthreads();
  const int rbase = (part * 4 + wave) * RBW;
  const int CB = (ncols + 15) / 16;
  const T *hp = a.Ht + ((int64_t)cell * a.RB) * a.KS * 64 + lane;

  T a0[4][RBW], a1[4][RBW];
  acc_t acc[RBW][CBM];
#pragma unroll
  for (int r = 0; r < RBW; ++r)
#pragma unroll
    for (int cb = 0; cb < CBM; ++cb) acc[r][cb] = (acc_t){0, 0, 0, 0};

  // Loads are unconditional, at clamped addresses, and nothing consumes a
  // loaded value before it is needed, so the compiler waits only for the
  // current chunk's operands and the next chunk's loads stay in flight.
  // Out-of-range rows and columns are zeroed when they are written to LDS
  // (row scale 0); a clamped A fragment then multiplies zero rows of Xs (k
  // past the end) or feeds accumulators that are never stored (row blocks
  // past the end).  Wide tiles read the rows as pairs of doubles with 32-bit
  // element offsets (even leading dimensions; the host checks the offsets fit).
  constexpr bool PAIRS = NC >= 32;
  constexpr int NP = PAIRS ? NC / 2 : NC, EPT2 = KC * NP / 256;
  static_assert(KC * NP % 256 == 0, "the gather must cover the chunk exactly");
  const int NPV = (ncols + 1) / 2;
  double2 xr[EPT2];
  auto stage_load = [&](int ch) {
    const uint32_t ld = (uint32_t)a.ldx;
#pragma unroll
    for (int j = 0; j < EPT2; ++j) {
      const int idx = t + 256 * j, r = idx / NP, cp = idx % NP;
      const uint32_t row = (uint32_t)gs[ch * KC + r];
      if constexpr (PAIRS) {
        xr[j] = *reinterpret_cast<const double2 *>(a.X + row * ld +
                                                   2u * (uint32_t)min(cp, NPV - 1));
      } else {
        xr[j].x = a.X[(int64_t)row * ld + min(cp, ncols - 1)];
      }
    }
  };
  auto stage_store = [&](int buf, int ch) {
#pragma unroll
    for (int j = 0; j < EPT2; ++j) {
      const int idx = t + 256 * j, r = idx / NP, cp = idx % NP;
      const double s = gsc[ch * KC + r];
      if constexpr (PAIRS) {
        Xs[buf][r][2 * cp] = 2 * cp < ncols ? (T)(s * xr[j].x) : (T)0;
        Xs[buf][r][2 * cp + 1] = 2 * cp + 1 < ncols ? (T)(s * xr[j].y) : (T)0;
      } else {
        Xs[buf][r][cp] = cp < ncols ? (T)(s * xr[j].x) : (T)0;
      }
    }
  };
  auto a_load = [&](int ch, T (&dst)[4][RBW]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int r = 0; r < RBW; ++r) {
        const int64_t rb = min(rbase + r, a.RB - 1);
        dst[s][r] = ld_nt(&hp[(rb * a.KS + min(4 * ch + s, a.KS - 1)) * 64]);
      }
  };
  auto compute = [&](int buf, const T (&src)[4][RBW]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      T bv[CBM];
#pragma unroll
      for (int cb = 0; cb < CBM; ++cb) bv[cb] = Xs[buf][s * 4 + lk][cb * 16 + li];
#pragma unroll
      for (int r = 0; r < RBW; ++r)
#pragma unroll
        for (int cb = 0; cb < CBM; ++cb) acc[r][cb] = M::op(src[s][r], bv[cb], acc[r][cb]);
    }
  };
  auto step = [&](int ch, const T (&cur)[4][RBW], T (&nxt)[4][RBW], int buf) {
    const bool more = ch + 1 < NCH;
    if (more) {
      stage_load(ch + 1);
      a_load(ch + 1, nxt);
    }
    compute(buf, cur);
    if (more) stage_store(buf ^ 1, ch + 1);
    __syncthreads();
  };

  stage_load(0);
  a_load(0, a0);
  stage_store(0, 0);
  __syncthreads();
  for (int ch = 0; ch < NCH; ch += 2) {
    step(ch, a0, a1, 0);
    if (ch + 1 < NCH) step(ch + 1, a1, a0, 1);
  }
  // scatter: per row block, all reads of Y first, then all writes, so the
  // reads overlap instead of each waiting for the one before; the wide tiles
  // stream Y non-temporally (the narrow ones, whose rows are a 128-byte
  // piece, measured slower that way)
  constexpr bool YNT = CBM > 1;
#pragma unroll
  for (int r = 0; r < RBW; ++r) {
    const int rb = rbase + r;
    if (rb >= a.RB) continue;
    int64_t node[4];
    bool ok[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = rb * 16 + M::row(v, lk);
      node[v] = gs[min(row, nloc - 1)];
      ok[v] = row < nloc;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) ok[v] = ok[v] && a.minv[node[v]] != 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double yv[CBM];
#pragma unroll
      for (int cb = 0; cb < CBM; ++cb) {
        const int64_t o = node[v] * a.ldy + min(cb * 16 + li, ncols - 1);
        yv[cb] = YNT ? ld_nt(&a.Y[o]) : a.Y[o];
      }
#pragma unroll
      for (int cb = 0; cb < CBM; ++cb) {
        const int col = cb * 16 + li;
        if (ok[v] && cb < CB && col < ncols) {
          const double y = yv[cb] + a.alpha * (double)acc[r][cb][v];
          if (YNT)
            st_nt(y, &a.Y[node[v] * a.ldy + col]);
          else
            a.Y[node[v] * a.ldy + col] = y;
        }
      }
    }
  }
}

// BF16 variant: v_mfma_f32_16x16x32_bf16, FP32 accumulation.  A operand tile
// [cell][rb][ks32][lane][8]: lane l holds H[16 rb + l%16][32 ks + 8 (l/16) + e];
// the gathered block is kept transposed in LDS (XT[col][k]) so that the eight
// k values of a B operand are one 16-byte read.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

__device__ inline __bf16 to_bf16(double x) { return (__bf16)(float)x; }

template <int NT>
__global__ __launch_bounds__(256) void k_cell_bf16(int ncells, int ntiles,
                                                   const int32_t *__restrict__ cells,
                                                   const int32_t *__restrict__ c2g, int nloc,
                                                   int RB, int KS32, const v8bf *__restrict__ Ht,
                                                   const double *__restrict__ Xh, int64_t ldx,
                                                   const double *__restrict__ scale,
                                                   double *__restrict__ Y, int64_t ldy,
                                                   const double *__restrict__ minv, int ncols,
                                                   double alpha) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int KP = KS32 * 32;
  const int SK = KP + 8;                   // row stride of XT in bf16 elements
  __bf16 *XT = (__bf16 *)smem;             // [NT][SK]
  const int b = blockIdx.x;
  const int xcd = b % 8, slot = b / 8;
  const int ci = (slot / ntiles) * 8 + xcd;
  const int tile = slot % ntiles;
  if (ci >= ncells) return;
  const int cell = cells[ci];
  const int col0 = tile * NT;
  const int32_t *g = c2g + (int64_t)cell * nloc;
  for (int idx = threadIdx.x; idx < KP * NT; idx += 256) {
    const int r = idx / NT, cc = idx % NT;
    double v = 0.0;
    if (r < nloc && col0 + cc < ncols) {
      const int64_t node = g[r];
      const double s = minv[node] == 0.0 ? 0.0 : (scale ? scale[node] : 1.0);
      v = s * Xh[node * ldx + col0 + cc];
    }
    XT[cc * SK + r] = to_bf16(v);
  }
  __syncthreads();
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int li = lane % 16, lk = lane / 16;
  for (int rb = wave; rb < RB; rb += 4) {
    v4f acc[NT / 16];
    for (int cb = 0; cb < NT / 16; ++cb) acc[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
    const v8bf *hp = Ht + (((int64_t)cell * RB + rb) * KS32) * 64 + lane;
    for (int ks = 0; ks < KS32; ++ks) {
      const v8bf a = hp[(int64_t)ks * 64];
#pragma unroll
      for (int cb = 0; cb < NT / 16; ++cb) {
        const v8bf bv = *(const v8bf *)(XT + (cb * 16 + li) * SK + ks * 32 + lk * 8);
        acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bv, acc[cb], 0, 0, 0);
      }
    }
    for (int v = 0; v < 4; ++v) {
      const int row = rb * 16 + 4 * lk + v;
      if (row >= nloc) continue;
      const int64_t node = g[row];
      if (minv[node] == 0.0) continue;
#pragma unroll
      for (int cb = 0; cb < NT / 16; ++cb) {
        const int col = col0 + cb * 16 + li;
        if (col < ncols) Y[node * ldy + col] += alpha * (double)acc[cb][v];
      }
    }
  }
}


// Affine epilogue of an apply (device copy of ApplyEpilogue)
struct EpiArgs {
  double alpha, beta, gamma;
  const double *Z1, *Z2, *G, *Cl;
};
// Affine epilogue terms of one element: beta Z1 + gamma Z2 + alpha G Cl
__device__ inline double epi_terms(const EpiArgs &e, int64_t o, int col) {
  double v = 0.0;
  if (e.Z1) v += e.beta * e.Z1[o];
  if (e.Z2) v += e.gamma * e.Z2[o];
  if (e.G) v += e.alpha * e.G[o] * e.Cl[col];
  return v;
}

// ------------------------------------------------------------------ coupling
// Column of column block cb and lane li in the wide tiles: a lane's blocks 2q
// and 2q + 1 are adjacent columns, so its operands come from LDS as one pair
// and its results go to memory as 16-byte pairs.  A single block (CBM = 1, up
// to 16 vectors) keeps the plain order.
template <int CBM>
__device__ __forceinline__ int tile_col(int cb, int li) {
  return CBM == 1 ? li : 32 * (cb / 2) + 2 * li + (cb & 1);
}

// 16 rows x 16 CBM columns of an operand block on their way to LDS: thread t
// carries pairs t, t + 256, ... (CBM = 1: one element).  Rows come from
// `base` at row numbers in LDS; `vec`: even ld and 16-byte aligned rows.
template <typename T, int CBM>
struct RowStage {
  static constexpr int NC = 16 * CBM, NP = NC / 2, E = CBM == 1 ? 1 : 16 * NP / 256;
  static_assert(CBM == 1 || 16 * NP % 256 == 0, "the rows must be covered exactly");
  double2 x[E];
  __device__ __forceinline__ void load(const double *base, int64_t ld, const int32_t *rows,
                                       int ncols, bool vec) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int idx = threadIdx.x + 256 * j;
      if constexpr (CBM == 1) {
        x[j].x = base[rows[idx / 16] * ld + min(idx % 16, ncols - 1)];
      } else {
        const double *r = base + rows[idx / NP] * ld;
        const int c = 2 * (idx % NP);
        if (vec) {
          x[j] = *reinterpret_cast<const double2 *>(r + min(c, (ncols - 1) & ~1));
        } else {
          x[j].x = r[min(c, ncols - 1)];
          x[j].y = r[min(c + 1, ncols - 1)];
        }
      }
    }
  }
  // scale (may be NULL: 1) per row; a zero drops the row
  __device__ __forceinline__ void store(T *Xs, const double *scale) const {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int idx = threadIdx.x + 256 * j;
      const int r = CBM == 1 ? idx / 16 : idx / NP;
      const double s = scale ? scale[r] : 1.0;
      const T vx = s != 0.0 ? (T)(s * x[j].x) : (T)0;
      if constexpr (CBM == 1) {
        Xs[idx] = vx;
      } else {
        const T vy = s != 0.0 ? (T)(s * x[j].y) : (T)0;
        Xs[r * NC + 2 * (idx % NP)] = vx;
        Xs[r * NC + 2 * (idx % NP) + 1] = vy;
      }
    }
  }
};

// acc += (16 x 4 operand fragment a of k step s) (rows 4 s .. of the chunk)
template <typename T, int CBM, typename Acc>
__device__ __forceinline__ void tile_step(const T *Xs, int s, T a, int li, int lk, Acc (&acc)[CBM]) {
  typedef T T2 __attribute__((ext_vector_type(2)));
  const T *row = Xs + (4 * s + lk) * 16 * CBM;
  if constexpr (CBM == 1) {
    acc[0] = CellMfma<T>::op(a, row[li], acc[0]);
  } else {
    T2 b[CBM / 2];
#pragma unroll
    for (int q = 0; q < CBM / 2; ++q) b[q] = *reinterpret_cast<const T2 *>(row + 32 * q + 2 * li);
#pragma unroll
    for (int q = 0; q < CBM / 2; ++q) {
      acc[2 * q] = CellMfma<T>::op(a, b[q].x, acc[2 * q]);
      acc[2 * q + 1] = CellMfma<T>::op(a, b[q].y, acc[2 * q + 1]);
    }
  }
}

// blocks of one set of functions (couple.hip) as the kernels take them
template <typename T>
struct BoxSet {
  const int32_t *ptr, *rboff, *rbbox, *atom;
  const int64_t *ksoff;
  const T *tile;
  const uint32_t *live;
  int nf;
};

// Yp = [E ; P^C] (s X^C) box by box: one partial row per (box, function).  A
// work-group takes four 16-row blocks of a box (couple.hip orders them E first,
// then P^C), one a wave, and all columns; the box's 512 nodes stream through
// LDS in 16-row chunks, double buffered, while the next chunk's rows and matrix
// fragments are on their way in registers.  Bound by the FP64 matrix cores at
// 160 vectors, which counters find busy 49% of the time (64 atoms: 0.85 ms, 3.9 GB
// through HBM, 4.6 TB/s; 500 atoms 57%); two waves a SIMD without spills beat three
// with 21 spilled registers and every chunk multiplied, 1.23 ms.  Bound by reading
// the blocks at one vector.
template <typename T>
struct GatherArgs {
  const int32_t *items;
  const double *X, *minv;
  int64_t ldx, ldp, prow;          // prow: first partial row of the projectors
  int64_t nre, nrk;                // 16-row blocks of E and P^C in the list
  double *Yp;
  BoxSet<T> E;
  BoxSet<double> K;
  NodeGrid g;
  int ncols;
  bool scaled, vec;
};

template <typename T, int CBM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CBM > 8 ? 2 : 3)))
void k_box_gather(GatherArgs<T> a) {
  typedef CellMfma<T> M;
  typedef typename M::acc_t acc_t;
  constexpr int NB = EFE_BOX * EFE_BOX * EFE_BOX, KS = NB / 4, NCH = NB / 16;
  __shared__ __align__(16) T Xs[2][16 * 16 * CBM];
  __shared__ int32_t gs[NB];
  __shared__ double gsc[NB];
  int64_t blk = blockIdx.x;        // the parts of a box run on one XCD
  if (gridDim.x % 8 == 0) blk = (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int box = a.items[2 * blk];
  const int t = threadIdx.x, wave = t / 64, lane = t % 64, li = lane % 16, lk = lane / 16;
  const int r0 = a.items[2 * blk + 1];
  const int ne = a.E.rboff[box + 1] - a.E.rboff[box], nk = a.K.rboff[box + 1] - a.K.rboff[box];
  // with T = float only E blocks are listed; with T = double both layouts are
  // the same.  A wave past the last block repeats the first one's loads.
  // Which wave (SIMD) is left over turns with the work-group.
  const int rw = r0 + (wave + (int)blockIdx.x / 8) % 4;
  const bool work = rw < ne + (sizeof(T) == 8 ? nk : 0);
  const int r = work ? rw : r0;
  const bool isE = r < ne;
  int o[3], ijk[3];
  box_origin(a.g, EFE_BOX, box, o);
  for (int i = t; i < NB; i += 256) {
    const bool in = box_node(a.g, EFE_BOX, o, i, ijk);
    const int32_t node = in ? ijk[0] + a.g.n1[0] * (ijk[1] + a.g.n1[1] * ijk[2]) : 0;
    gs[i] = node;
    gsc[i] = in ? (a.scaled ? a.minv[node] : 1.0) : 0.0;
  }
  __syncthreads();
  const T *tp = (isE ? a.E.tile + (int64_t)(a.E.rboff[box] + r) * KS * 64
                     : (const T *)a.K.tile + (int64_t)(a.K.rboff[box] + r - ne) * KS * 64) +
                lane;
  // chunks whose entries are not all zero (a box reaches beyond the atoms' cells)
  static_assert(NCH == 32, "one bit per chunk");
  const uint32_t live = work ? __builtin_amdgcn_readfirstlane(
                                   isE ? a.E.live[a.E.rboff[box] + r] : a.K.live[a.K.rboff[box] + r - ne])
                             : 0u;
  acc_t acc[CBM];
#pragma unroll
  for (int cb = 0; cb < CBM; ++cb) acc[cb] = (acc_t){0, 0, 0, 0};
  RowStage<T, CBM> st;
  T a0[4], a1[4];
  auto a_load = [&](int ch, T (&d)[4]) {
    if (live >> ch & 1)
#pragma unroll
      for (int s = 0; s < 4; ++s) d[s] = ld_nt(tp + (4 * ch + s) * 64);
  };
  auto step = [&](int ch, const T (&cur)[4], T (&nxt)[4], int buf) {
    if (ch + 1 < NCH) {
      st.load(a.X, a.ldx, gs + 16 * (ch + 1), a.ncols, a.vec);
      a_load(ch + 1, nxt);
    }
    if (live >> ch & 1)
#pragma unroll
      for (int s = 0; s < 4; ++s) tile_step<T, CBM>(Xs[buf], s, cur[s], li, lk, acc);
    if (ch + 1 < NCH) st.store(Xs[buf ^ 1], gsc + 16 * (ch + 1));
    __syncthreads();
  };
  st.load(a.X, a.ldx, gs, a.ncols, a.vec);
  a_load(0, a0);
  st.store(Xs[0], gsc);
  __syncthreads();
  // FP32 sums run over one brick (64 nodes) and are added up in FP64: the terms
  // of E s X^C cancel, so rounding the running sum over all 512 nodes cost more
  // than rounding the operands (filter error 7.0e-5 against 4.2e-5)
  v4d sum[sizeof(T) == 4 ? CBM : 1];
  if constexpr (sizeof(T) == 4)
#pragma unroll
    for (int cb = 0; cb < CBM; ++cb) sum[cb] = (v4d){0.0, 0.0, 0.0, 0.0};
  for (int ch = 0; ch < NCH; ch += 4) {
    step(ch, a0, a1, 0);
    step(ch + 1, a1, a0, 1);
    step(ch + 2, a0, a1, 0);
    step(ch + 3, a1, a0, 1);
    if constexpr (sizeof(T) == 4) {
      if (live >> ch & 15)
#pragma unroll
        for (int cb = 0; cb < CBM; ++cb) {
#pragma unroll
          for (int v = 0; v < 4; ++v) sum[cb][v] += (double)acc[cb][v];
          acc[cb] = (acc_t){0, 0, 0, 0};
        }
    }
  }
  if (!work) return;
  const int nf = isE ? a.E.nf : 1, rb = isE ? r : r - ne;
  const int32_t *ptr = isE ? a.E.ptr : a.K.ptr;
  const int nrow = (ptr[box + 1] - ptr[box]) * nf;
  const int64_t row0 = (isE ? 0 : a.prow) + (int64_t)ptr[box] * nf;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int f = 16 * rb + M::row(v, lk);
    if (f >= nrow) continue;
    double *yp = a.Yp + (row0 + f) * a.ldp;
#pragma unroll
    for (int cb = 0; cb < CBM; ++cb) {
      const int col = tile_col<CBM>(cb, li);
      if (col >= a.ncols) continue;
      if constexpr (sizeof(T) == 4)
        st_nt(sum[cb][v], yp + col);
      else
        st_nt(acc[cb][v], yp + col);
    }
  }
}

// The same where k_box_gather has too few work-groups to hide its chain of
// chunks (GATHER_FEW): one work-group per 16-row block and 16 columns, one wave
// per 64 nodes (a brick) with all its operands requested at once, straight from
// memory; the eight sums meet in LDS in a fixed order.  27 boxes and 8 vectors:
// 7.1 us, 15.7 in chunks.
template <typename T>
__global__ __launch_bounds__(512) void k_box_gather_few(GatherArgs<T> a) {
  typedef CellMfma<T> M;
  typedef typename M::acc_t acc_t;
  constexpr int NB = EFE_BOX * EFE_BOX * EFE_BOX, KS = NB / 4, KW = KS / 8;
  __shared__ double red[8][256];
  const bool isE = (int64_t)blockIdx.x < a.nre;   // E blocks first, then P^C blocks
  const int64_t rb = isE ? blockIdx.x : blockIdx.x - a.nre;
  const int box = (isE ? a.E.rbbox : a.K.rbbox)[rb];
  const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t / 64), lane = t % 64;
  const int li = lane % 16, lk = lane / 16;
  const int c0 = (int)blockIdx.y * 16, col = min(c0 + li, a.ncols - 1);
  const uint32_t live = (isE ? a.E.live[rb] : a.K.live[rb]) >> (4 * wave) & 15;
  acc_t acc = (acc_t){0, 0, 0, 0};
  if (live) {
    const T *tp = (isE ? a.E.tile : (const T *)a.K.tile) + (rb * KS + wave * KW) * 64 + lane;
    int o[3], ijk[3];
    box_origin(a.g, EFE_BOX, box, o);
    T av[KW];
    double x[KW], m[KW];
#pragma unroll
    for (int s = 0; s < KW; ++s) {
      const bool in = box_node(a.g, EFE_BOX, o, 4 * (KW * wave + s) + lk, ijk);
      const int32_t node = in ? ijk[0] + a.g.n1[0] * (ijk[1] + a.g.n1[1] * ijk[2]) : 0;
      av[s] = tp[s * 64];
      x[s] = a.X[(int64_t)node * a.ldx + col];
      const double w = a.scaled ? a.minv[node] : 1.0;
      m[s] = in ? w : 0.0;
    }
#pragma unroll
    for (int s = 0; s < KW; ++s)
      if (live >> (s / 4) & 1)
        acc = M::op(av[s], m[s] != 0.0 ? (T)(m[s] * x[s]) : (T)0, acc);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][M::row(v, lk) * 16 + li] = (double)acc[v];
  __syncthreads();
  if (t >= 256 || c0 + t % 16 >= a.ncols) return;
  const int nf = isE ? a.E.nf : 1, f = 16 * (int)(rb - (isE ? a.E.rboff : a.K.rboff)[box]) + t / 16;
  const int32_t *ptr = isE ? a.E.ptr : a.K.ptr;
  if (f >= (ptr[box + 1] - ptr[box]) * nf) return;
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < 8; ++w) s += red[w][t];
  a.Yp[((isE ? 0 : a.prow) + (int64_t)ptr[box] * nf + f) * a.ldp + c0 + t % 16] = s;
}

// Coefficients of one apply, interleaved atom by atom: rows (I, k) of Q, k <
// nf the enrichment rows of the vectors (times the atom's block of
// (M~^ee)^-1 when inv is given), k = nf (with projectors) P^C_I s X^C; R = E s
// X^C.  One work-group per (atom, 64 columns), one wave per function; the
// partial rows of the atom's boxes are added in box order, sixteen in flight
// (four in flight left the sums waiting for memory: 105 us for 64 atoms and
// 160 vectors).
struct SumArgs {
  const int32_t *e_ptr, *e_pos, *k_ptr, *k_pos;
  const double *Yp, *XE, *inv;
  int64_t ldp, lde, ldq, prow;
  double *Q, *R;
  int nf, nx, ncols;
  // without enrichment the dense part is W = D P^C s X^C, done here (a launch of
  // 4.7 us less): D and the rows of W (else NULL)
  const double *D;
  double *W;
};

__global__ __launch_bounds__(640) void k_coef_sum(SumArgs a) {
  const int I = blockIdx.x;
  const int k = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64)), lane = threadIdx.x % 64;
  const bool isE = k < a.nf;
  const int col = blockIdx.y * 64 + lane, cc = min(col, a.ncols - 1);
  const int32_t *ptr = isE ? a.e_ptr : a.k_ptr, *pos = isE ? a.e_pos : a.k_pos;
  const int nf = isE ? a.nf : 1;
  const double *yp = a.Yp + ((isE ? 0 : a.prow) + (isE ? k : 0)) * a.ldp + cc;
  const int32_t q0 = ptr[I], q1 = ptr[I + 1];
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int32_t q = q0; q < q1; q += 16) {
    double v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j)
      v[j] = ld_nt(yp + (int64_t)pos[min(q + j, q1 - 1)] * nf * a.ldp);
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (q + j < q1) s[j % 4] += v[j];
  }
  const double sum = (s[0] + s[1]) + (s[2] + s[3]);
  if (col >= a.ncols) return;
  double *q = a.Q + ((int64_t)I * a.nx + k) * a.ldq + col;
  if (!isE) {
    *q = sum;
    if (a.D) a.W[I * a.ldq + col] = a.D[I] * sum;
    return;
  }
  a.R[((int64_t)I * a.nf + k) * a.ldq + col] = sum;
  const double *xe = a.XE + (int64_t)I * a.nf * a.lde + col;
  if (a.inv) {
    const double *m = a.inv + ((int64_t)I * a.nf + k) * a.nf;
    double x = 0.0;
    for (int l = 0; l < a.nf; ++l) x += m[l] * xe[l * a.lde];
    *q = x;
  } else {
    *q = xe[k * a.lde];
  }
}

// the same for up to 16 vectors: the lanes of a wave share the boxes out, and
// their sums meet in a fixed tree
__global__ __launch_bounds__(640) void k_coef_sum_narrow(SumArgs a, int cw) {
  const int I = blockIdx.x;
  const int k = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64)), lane = threadIdx.x % 64;
  const bool isE = k < a.nf;
  const int col = lane % cw, sl = lane / cw, nsl = 64 / cw, cc = min(col, a.ncols - 1);
  const int32_t *ptr = isE ? a.e_ptr : a.k_ptr, *pos = isE ? a.e_pos : a.k_pos;
  const int nf = isE ? a.nf : 1;
  const double *yp = a.Yp + ((isE ? 0 : a.prow) + (isE ? k : 0)) * a.ldp + cc;
  const int32_t q0 = ptr[I], q1 = ptr[I + 1];
  double sum = 0.0;
  for (int32_t q = q0 + sl; q < q1; q += 4 * nsl) {
    double v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = yp[(int64_t)pos[min(q + j * nsl, q1 - 1)] * nf * a.ldp];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (q + j * nsl < q1) sum += v[j];
  }
  for (int o = cw; o < 64; o <<= 1) sum += __shfl_xor(sum, o);
  if (lane >= a.ncols) return;   // sl = 0 and a column of the block
  double *q = a.Q + ((int64_t)I * a.nx + k) * a.ldq + col;
  if (!isE) {
    *q = sum;
    if (a.D) a.W[I * a.ldq + col] = a.D[I] * sum;
    return;
  }
  a.R[((int64_t)I * a.nf + k) * a.ldq + col] = sum;
  const double *xe = a.XE + (int64_t)I * a.nf * a.lde + col;
  if (a.inv) {
    const double *m = a.inv + ((int64_t)I * a.nf + k) * a.nf;
    double x = 0.0;
    for (int l = 0; l < a.nf; ++l) x += m[l] * xe[l * a.lde];
    *q = x;
  } else {
    *q = xe[k * a.lde];
  }
}

// Dense part: S Q with the symmetric matrix of the coefficients (couple.hip).
// Rows k < nf: Y^E = alpha (R + S Q) + epilogue terms; rows k = nf: the
// projector coefficients W, behind the rows of Q.  One work-group per 16 rows
// and 16 CB columns; its four waves take every fourth k step and their sums
// meet in LDS in a fixed order (the split of the sum over work-groups that this
// replaces needed a cleared output and atomics).
template <int CB>
__global__ __launch_bounds__(256) void k_coef_dense(int64_t n, int nf, int nx, int ncols,
                                                    const double *__restrict__ S, double *Q,
                                                    int64_t ldq, const double *__restrict__ R,
                                                    EpiArgs e, double *YE, int64_t ldy) {
  __shared__ double red[4][16][16 * CB];
  const int t = threadIdx.x, wave = t / 64, lane = t % 64, li = lane % 16, lk = lane / 16;
  const int64_t row0 = (int64_t)blockIdx.x * 16;
  const int c0 = blockIdx.y * 16 * CB;
  const int64_t rl = min(row0 + li, n - 1);
  int cc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) cc[cb] = min(c0 + 16 * cb + li, ncols - 1);
  v4d acc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) acc[cb] = (v4d){0.0, 0.0, 0.0, 0.0};
  const int64_t nks = (n + 3) / 4;
#pragma unroll 4
  for (int64_t ks = wave; ks < nks; ks += 4) {
    const int64_t kk = min(4 * ks + lk, n - 1);
    const double av = 4 * ks + lk < n ? S[kk * n + rl] : 0.0;
    double bv[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) bv[cb] = Q[kk * ldq + cc[cb]];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
      acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[cb], acc[cb], 0, 0, 0);
  }
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][4 * v + lk][16 * cb + li] = acc[cb][v];
  __syncthreads();
  for (int i = t; i < 256 * CB; i += 256) {
    const int rr = i / (16 * CB), c = i % (16 * CB), col = c0 + c;
    const int64_t row = row0 + rr;
    if (row >= n || col >= ncols) continue;
    const double v = (red[0][rr][c] + red[1][rr][c]) + (red[2][rr][c] + red[3][rr][c]);
    const int64_t I = row / nx;
    const int k = (int)(row - I * nx);
    if (k < nf) {
      const int64_t f = I * nf + k, o = f * ldy + col;
      YE[o] = e.alpha * (v + R[f * ldq + col]) + epi_terms(e, o, col);
    } else {
      Q[(n + I) * ldq + col] = v;
    }
  }
}

// All terms of Y^C but dense cell products:
//   Y^C = alpha (sum over the node's cells of Yc + E^T X^E + P^C^T W)
//         + beta Z1 + gamma Z2 + alpha G diag(Cl)      (boundary rows 0)
// brick by brick (4 x 4 x 4 nodes): each of the four waves multiplies 16 nodes
// (one z layer) by all columns, the coefficient rows of the brick's atoms
// streaming through LDS; the other terms are read and Y^C is written once, in
// 16-byte pieces.  HBM-bound: the products of one brick run while others
// wait for their rows (counters, 64 atoms, 160 vectors: 7.2 GB read and 1.2 GB
// written in 1.62 ms, 5.2 TB/s, matrix cores busy 22% of the time; 500 atoms 56 and
// 7.6 GB in 14.9 ms, 4.3 TB/s, 28%; the separate start-value pass and colour passes
// it replaces took 5.3 ms for 64 atoms).
template <typename T>
struct NodeArgs {
  BoxSet<T> E;
  BoxSet<double> K;
  const double *Q, *Yc;
  int64_t ldq, ldc, wrow;          // wrow: first row of W in Q
  int nx, ncols, nparts;           // nparts: column parts of 16 CBM
  NodeGrid g;
  EpiArgs e;
  double *Y;
  int64_t ldy;
  bool vec;
  int first;                       // first column of part 0
};

constexpr int NODE_SEG = 512;      // functions whose row numbers sit in LDS

// acc += tile (16 nodes x K functions) times the functions' rows of Q
template <typename T, int CBM, typename Acc>
__device__ __forceinline__ void brick_product(const T *tp, int K, const int32_t *atoms, int nf,
                                              int nx, int64_t row0, const double *Q, int64_t ldq,
                                              int ncols, T *Xs, int32_t *gs, Acc (&acc)[CBM]) {
  const int t = threadIdx.x, lane = t % 64, li = lane % 16, lk = lane / 16;
  for (int f0 = 0; f0 < K; f0 += NODE_SEG) {
    const int nseg = min(K - f0, NODE_SEG), KS = (nseg + 3) / 4, NCH = (nseg + 15) / 16;
    __syncthreads();
    for (int i = t; i < 16 * NCH; i += 256) {
      const int f = f0 + min(i, nseg - 1);
      gs[i] = (int32_t)(row0 + (int64_t)atoms[f / nf] * nx + f % nf);
    }
    __syncthreads();
    RowStage<T, CBM> st;
    T a0[4], a1[4];
    const T *sp = tp + (f0 / 4) * 64;
    auto a_load = [&](int ch, T (&d)[4]) {
#pragma unroll
      for (int s = 0; s < 4; ++s) d[s] = ld_nt(sp + min(4 * ch + s, KS - 1) * 64);
    };
    auto step = [&](int ch, const T (&cur)[4], T (&nxt)[4], int buf) {
      if (ch + 1 < NCH) {
        st.load(Q, ldq, gs + 16 * (ch + 1), ncols, true);
        a_load(ch + 1, nxt);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (4 * ch + s < KS)
          tile_step<T, CBM>(Xs + buf * 256 * CBM, s, cur[s], li, lk, acc);
      if (ch + 1 < NCH) st.store(Xs + (buf ^ 1) * 256 * CBM, nullptr);
      __syncthreads();
    };
    st.load(Q, ldq, gs, ncols, true);
    a_load(0, a0);
    st.store(Xs, nullptr);
    __syncthreads();
    for (int ch = 0; ch < NCH; ch += 2) {
      step(ch, a0, a1, 0);
      if (ch + 1 < NCH) step(ch + 1, a1, a0, 1);
    }
  }
}

// FEW (one column block): what the nodes add to the products is requested
// first, all of it at once, instead of cell after cell behind the products (17^3
// nodes and 8 vectors: 9.4 us, before 15.0).  With bricks enough to cover those
// waits the registers cost more (0.91 M nodes, one vector: 203 us against 175).
template <typename T, int CBM, bool FEW = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
void k_node_update(NodeArgs<T> a) {
  __shared__ __align__(16) double Xs[2 * 256 * CBM];
  __shared__ int32_t gs[NODE_SEG];
  // the column parts of a brick, and neighbouring bricks, run on one XCD
  int64_t b = blockIdx.x;
  if (gridDim.x % 8 == 0) b = (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int c0 = a.first + (int)(b % a.nparts) * 16 * CBM, ncols = min(a.ncols - c0, 16 * CBM);
  b /= a.nparts;
  const double *const Qc = a.Q + c0;
  const int t = threadIdx.x, wave = t / 64, lane = t % 64, li = lane % 16, lk = lane / 16;
  const NodeGrid &g = a.g;
  double pre[FEW ? 4 : 1][9];
  if constexpr (FEW) {
    static_assert(CBM == 1, "the wide tiles read their terms in pairs");
    int o[3];
    box_origin(g, EFE_BRICK, b, o);
    const int gi = o[0] + lk, gk = o[2] + wave;
    const int cx = gi / g.p, cz = gk / g.p, lx = gi - cx * g.p, lz = gk - cz * g.p;
    const bool inxz = gi > 0 && gi < g.n1[0] - 1 && gk > 0 && gk < g.n1[2] - 1;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int gj = o[1] + v, cy = gj / g.p, ly = gj - cy * g.p;
#pragma unroll
      for (int n = 0; n < 9; ++n) pre[v][n] = 0.0;
      if (!inxz || gj <= 0 || gj >= g.n1[1] - 1 || li >= ncols) continue;
      if (a.Yc)
#pragma unroll
        for (int n = 0; n < 8; ++n) {
          const int x = n & 1, y = n >> 1 & 1, z = n >> 2;
          if ((x && lx) || (y && ly) || (z && lz)) continue;
          const int64_t cell = cx - x + g.nc[0] * (cy - y + (int64_t)g.nc[1] * (cz - z));
          const int l = (x ? g.p : lx) + g.P * ((y ? g.p : ly) + g.P * (z ? g.p : lz));
          pre[v][n] = a.Yc[(cell * (g.P * g.P * g.P) + l) * a.ldc + c0 + li];
        }
      const int64_t row = ((int64_t)gi + (int64_t)g.n1[0] * (gj + (int64_t)g.n1[1] * gk)) * a.ldy + c0;
      pre[v][8] = epi_terms(a.e, row + li, c0 + li);
    }
  }
  v4d acc[CBM];
#pragma unroll
  for (int cb = 0; cb < CBM; ++cb) acc[cb] = (v4d){0.0, 0.0, 0.0, 0.0};
  {
    const int a0 = a.E.ptr[b], K = (a.E.ptr[b + 1] - a0) * a.E.nf;
    if (K > 0) {
      const T *tp = a.E.tile + 256 * a.E.ksoff[b] + (int64_t)wave * ((K + 3) / 4) * 64 + lane;
      if constexpr (sizeof(T) == 8) {
        brick_product<T, CBM>(tp, K, a.E.atom + a0, a.E.nf, a.nx, 0, Qc, a.ldq, ncols, Xs, gs,
                              acc);
      } else {
        v4f acf[CBM];
#pragma unroll
        for (int cb = 0; cb < CBM; ++cb) acf[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
        brick_product<T, CBM>(tp, K, a.E.atom + a0, a.E.nf, a.nx, 0, Qc, a.ldq, ncols, (T *)Xs,
                              gs, acf);
        // the FP32 blocks hold their rows so that both accumulator layouts agree
#pragma unroll
        for (int cb = 0; cb < CBM; ++cb)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[cb][v] = (double)acf[cb][v];
      }
    }
  }
  {
    const int a0 = a.K.ptr[b], K = a.K.ptr[b + 1] - a0;
    if (K > 0) {
      const double *tp = a.K.tile + 256 * a.K.ksoff[b] + (int64_t)wave * ((K + 3) / 4) * 64 + lane;
      brick_product<double, CBM>(tp, K, a.K.atom + a0, 1, 1, a.wrow, Qc, a.ldq, ncols, Xs, gs,
                                 acc);
    }
  }
  // accumulator v of lane l: node 4 v + l/16 of the layer, i.e. (x, y) = (l/16, v)
  int o[3];
  box_origin(g, EFE_BRICK, b, o);
  const int gi = o[0] + lk, gk = o[2] + wave;
  if (gi >= g.n1[0] || gk >= g.n1[2]) return;
  const EpiArgs &e = a.e;
  const int cx = gi / g.p, cz = gk / g.p, lx = gi - cx * g.p, lz = gk - cz * g.p;
  constexpr int NQ = CBM == 1 ? 1 : CBM / 2;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int gj = o[1] + v;
    if (gj >= g.n1[1]) break;
    const int64_t row = ((int64_t)gi + (int64_t)g.n1[0] * (gj + (int64_t)g.n1[1] * gk)) * a.ldy + c0;
    const bool inner = gi > 0 && gi < g.n1[0] - 1 && gj > 0 && gj < g.n1[1] - 1 && gk > 0 &&
                       gk < g.n1[2] - 1;
    if constexpr (FEW) {
      if (li >= ncols) continue;
      double s = acc[0][v];   // the cells in the order of their numbers
#pragma unroll
      for (int n = 7; n >= 0; --n) s += pre[v][n];
      a.Y[row + li] = inner ? e.alpha * s + pre[v][8] : 0.0;
    } else if constexpr (CBM == 1) {
      if (li >= ncols) continue;
      double s = acc[0][v];
      if (a.Yc && inner) {
        const int cy = gj / g.p, ly = gj - cy * g.p;
        for (int z = lz == 0 ? -1 : 0; z <= 0; ++z)
          for (int y = ly == 0 ? -1 : 0; y <= 0; ++y)
            for (int x = lx == 0 ? -1 : 0; x <= 0; ++x) {
              const int64_t cell = cx + x + g.nc[0] * (cy + y + (int64_t)g.nc[1] * (cz + z));
              const int l = (x ? g.p : lx) + g.P * ((y ? g.p : ly) + g.P * (z ? g.p : lz));
              s += a.Yc[(cell * (g.P * g.P * g.P) + l) * a.ldc + c0 + li];
            }
      }
      const double terms = epi_terms(e, row + li, c0 + li);
      a.Y[row + li] = inner ? e.alpha * s + terms : 0.0;
    } else {
      // pairs by 16-byte accesses when the layout allows it (vec: even ld,
      // aligned arrays), else element by element
      auto ld2 = [&](const double *p, int q) -> double2 {
        const int c = 32 * q + 2 * li;
        if (a.vec && c + 1 < ncols) return ld_nt2(p + row + c);
        double2 r;
        r.x = c < ncols ? p[row + c] : 0.0;
        r.y = c + 1 < ncols ? p[row + c + 1] : 0.0;
        return r;
      };
      double2 z1[NQ], z2[NQ], gg[NQ], s[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        z1[q] = z2[q] = gg[q] = make_double2(0.0, 0.0);
        if (e.Z1) z1[q] = ld2(e.Z1, q);
        if (e.Z2) z2[q] = ld2(e.Z2, q);
        if (e.G) gg[q] = ld2(e.G, q);
        s[q] = make_double2(acc[2 * q][v], acc[2 * q + 1][v]);
      }
      if (a.Yc && inner) {
        const int cy = gj / g.p, ly = gj - cy * g.p;
        for (int z = lz == 0 ? -1 : 0; z <= 0; ++z)
          for (int y = ly == 0 ? -1 : 0; y <= 0; ++y)
            for (int x = lx == 0 ? -1 : 0; x <= 0; ++x) {
              const int64_t cell = cx + x + g.nc[0] * (cy + y + (int64_t)g.nc[1] * (cz + z));
              const int l = (x ? g.p : lx) + g.P * ((y ? g.p : ly) + g.P * (z ? g.p : lz));
              const double *yc = a.Yc + (cell * (g.P * g.P * g.P) + l) * a.ldc + c0 + 2 * li;
              double2 y2[NQ];
#pragma unroll
              for (int q = 0; q < NQ; ++q)
                y2[q] = 32 * q + 2 * li < ncols ? ld_nt2(yc + 32 * q) : make_double2(0.0, 0.0);
#pragma unroll
              for (int q = 0; q < NQ; ++q) {
                s[q].x += y2[q].x;
                s[q].y += y2[q].y;
              }
            }
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int c = 32 * q + 2 * li;
        if (c >= ncols) continue;
        const bool two = c + 1 < ncols;
        double2 y = make_double2(0.0, 0.0);
        if (inner) {
          const double cl0 = e.G ? e.Cl[c0 + c] : 0.0, cl1 = e.G && two ? e.Cl[c0 + c + 1] : 0.0;
          y.x = e.alpha * (s[q].x + gg[q].x * cl0) + e.beta * z1[q].x + e.gamma * z2[q].x;
          y.y = e.alpha * (s[q].y + gg[q].y * cl1) + e.beta * z1[q].y + e.gamma * z2[q].y;
        }
        if (a.vec && two) {
          st_nt2(y, a.Y + row + c);
        } else {
          a.Y[row + c] = y.x;
          if (two) a.Y[row + c + 1] = y.y;
        }
      }
    }
  }
}

// ------------------------------------------------------------------ overlap
// CFE rows: Y = w X (w = m or 1/m, zero on the boundary)
__global__ void k_rowscale(int64_t n, int ncols, const double *__restrict__ w,
                           const double *__restrict__ X, int64_t ldx, double *__restrict__ Y,
                           int64_t ldy) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= n * ncols) return;
  const int64_t r = idx / ncols, c = idx % ncols;
  Y[r * ldy + c] = w[r] * X[r * ldx + c];
}

// Enrichment rows: Y_I = inv_I X_I for each atom block
__global__ void k_enr_block_apply(int natoms, int nf, int ncols, const double *__restrict__ inv,
                                  const double *__restrict__ X, int64_t ldx,
                                  double *__restrict__ Y, int64_t ldy) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= (int64_t)natoms * nf * ncols) return;
  const int c = idx % ncols;
  const int64_t f = idx / ncols;
  const int I = f / nf, k = f % nf;
  const double *a = inv + ((int64_t)I * nf + k) * nf;
  double acc = 0.0;
  for (int l = 0; l < nf; ++l) acc += a[l] * X[((int64_t)I * nf + l) * ldx + c];
  Y[f * ldy + c] = acc;
}

// ------------------------------------------------------------------ launchers
// Colour passes of the dense cell GEMM in column chunks of 16 CBM.
template <typename T, int RBW, int CBM>
static void launch_cell3(efe_ctx *c, const T *Ht, const double *X, int64_t ldx,
                         const double *scale, double *Y, int64_t ldy, double alpha, int ncols) {
  CellOps<T> a;
  a.nparts = (int)cdiv(c->RB, 4 * RBW);
  a.c2g = c->d_c2g;
  a.nloc = c->nloc;
  a.RB = c->RB;
  a.KS = c->KS;
  a.Ht = Ht;
  a.ldx = ldx;
  a.scale = scale;
  a.minv = c->d_minv;
  a.ldy = ldy;
  a.alpha = alpha;
  for (int col0 = 0; col0 < ncols; col0 += 16 * CBM) {
    a.ncols = std::min(16 * CBM, ncols - col0);
    a.X = X + col0;
    a.Y = Y + col0;
    for (int col = 0; col < 8; ++col) {
      const int nc = c->colour_offsets[col + 1] - c->colour_offsets[col];
      if (nc == 0) continue;
      a.ncells = nc;
      a.cells = c->d_colour_order + c->colour_offsets[col];
      const int64_t nblk = cdiv(nc, 8) * 8 * a.nparts;
      const int t = efe_timer_begin(c, CBM == 1 ? EFE_T_CELL_NARROW : EFE_T_CELL);
      k_cell3<T, RBW, CBM><<<nblk, 256, 0, c->stream>>>(a);
      efe_timer_end(c, CBM == 1 ? EFE_T_CELL_NARROW : EFE_T_CELL, t);
    }
  }
}

// X -> Xc with an even leading dimension (the dense cell GEMM's paired gathers)
__global__ void k_copy_cols(int64_t rows, int ncols, const double *__restrict__ X, int64_t ldx,
                            double *__restrict__ Y, int64_t ldy) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= rows * ncols) return;
  const int64_t r = idx / ncols;
  const int j = (int)(idx % ncols);
  Y[r * ldy + j] = X[r * ldx + j];
}

template <typename T>
static BoxSet<T> box_set(const CoupleSet &S, bool brick, const T *tile) {
  return {brick ? S.d_bk_ptr : S.d_bx_ptr, S.d_rboff, S.d_rbbox, S.d_bk_atom, S.d_bk_off, tile, S.d_live, S.nf};
}

// column blocks of the register tile: the narrowest that holds the columns
// (the products of empty columns cost as much as those of full ones)
static int tile_blocks(int ncols) {
  const int n = (int)cdiv(ncols, 16);
  return n == 1 ? 1 : (n + 1) / 2 * 2;
}

// Few work-groups (small meshes) leave the chip waiting on one chain of loads
// each; 16-column parts make more of them, with shorter chains, and the blocks
// that the parts read again are in the caches.  FEW_GROUPS is two work-groups a
// CU.
constexpr int64_t FEW_GROUPS = 512;

// The gather in 16-column parts takes a time that grows with its work-groups, the
// chunked one at least its chain of 32 chunks.  Coefficients of an apply (gather,
// sums, dense part) in parts and in chunks, by work-groups: 920 (projectors only,
// 160 vectors) 26 and 70 us, 1,390 46 and 50, 1,759 54 and 63, 2,085 55 and 55,
// 2,146 76 and 73, 2,612 78 and 69, 13,060 230 and 142.
constexpr int64_t GATHER_FEW = 2048;

template <typename T>
static void launch_box_gather(efe_ctx *c, const GatherArgs<T> &a, int64_t n) {
  if (n == 0) return;
  if ((a.nre + a.nrk) * cdiv(a.ncols, 16) <= GATHER_FEW) {
    k_box_gather_few<T><<<dim3(a.nre + a.nrk, cdiv(a.ncols, 16)), 512, 0, c->stream>>>(a);
    return;
  }
#define GO(B) k_box_gather<T, B><<<n, 256, 0, c->stream>>>(a)
  switch (tile_blocks(a.ncols)) {
    case 1: GO(1); break;
    case 2: GO(2); break;
    case 4: GO(4); break;
    case 6: GO(6); break;
    case 8: GO(8); break;
    default: GO(10);
  }
#undef GO
}

template <typename T>
static void launch_node_update(efe_ctx *c, NodeArgs<T> a, const T *tile) {
  a.E = box_set(c->cpl_e, true, tile);
  a.K = box_set<double>(c->cpl_k, true, c->cpl_k.d_T1);
  // 64-column parts: their 95 registers leave five waves a SIMD to cover the
  // reads (64 atoms, 160 vectors: 1.61 ms, against 1.71 in 32-column parts, 1.9
  // in one 160-column part with two waves)
  const bool few = c->cpl_e.n_brick * cdiv(a.ncols, 64) < 2 * FEW_GROUPS;
  if (few) {
    a.nparts = (int)cdiv(a.ncols, 16);
    k_node_update<T, 1, true><<<c->cpl_e.n_brick * a.nparts, 256, 0, c->stream>>>(a);
    return;
  }
  // what is left of 64-column parts goes on its own in the narrowest tile that
  // holds it (500 atoms, 160 vectors: 14.9 ms, 15.9 as a third 64-column part
  // whose products are half empty; 64 atoms 1.62, 1.64)
  for (a.first = 0; a.first < a.ncols; a.first += 64 * a.nparts) {
    const int left = a.ncols - a.first, B = std::min(tile_blocks(left), 4);
    a.nparts = std::max(left / 64, 1);
    const int64_t n = c->cpl_e.n_brick * a.nparts;
    switch (B) {
      case 1: k_node_update<T, 1><<<n, 256, 0, c->stream>>>(a); break;
      case 2: k_node_update<T, 2><<<n, 256, 0, c->stream>>>(a); break;
      default: k_node_update<T, 4><<<n, 256, 0, c->stream>>>(a);
    }
  }
}

efe_status efe_apply_H_internal(efe_ctx *c, const double *XC, int64_t ldx, bool minv,
                                const double *XE, int64_t lde, double *Y, int64_t ldy, int ncols,
                                int prec, const ApplyEpilogue *epi) {
  if (!c->have_potential) EFE_FAIL(c, EFE_ESTATE, "no potential set");
  if (ncols <= 0) return EFE_OK;
  if (ncols > EFE_COL_CHUNK) EFE_FAIL(c, EFE_EINVAL, "apply chunk wider than 160 columns");
  if ((prec == EFE_FP32 && !c->have32) || (prec == EFE_BF16 && !c->have16))
    EFE_FAIL(c, EFE_ESTATE, "reduced-precision cell matrices were not built by efe_set_potential");
  if (prec == EFE_BF16 && c->n_enr > 0)
    EFE_FAIL(c, EFE_EINVAL, "the BF16 cell GEMM takes plain CFE systems only");
  efe_status s;
  const int64_t nn = c->n_nodes;
  ApplyEpilogue E0;
  const ApplyEpilogue &ep = epi ? *epi : E0;
  auto al = [](const double *p) { return p == nullptr || (uintptr_t)p % 16 == 0; };
  const bool xvec = ldx % 2 == 0 && al(XC);
  if ((!xvec || nn * ldx >= (1ll << 31)) && nn * (int64_t)((ncols + 1) & ~1) >= (1ll << 31))
    EFE_FAIL(c, EFE_EINVAL, "n_nodes x columns exceeds the 32-bit offsets of the cell GEMM");
  const bool tp = c->tp && prec != EFE_BF16;
  const double *scale = minv ? c->d_minv : nullptr;
  const double *Xd = XC;             // rows as the dense cell GEMM takes them
  int64_t ldd = ldx;
  if (!tp && (!xvec || nn * ldx >= (1ll << 31))) {
    double *Xc;
    ldd = (ncols + 1) & ~1;
    if ((s = efe_ws(c, 0, (size_t)nn * ldd * 8, (void **)&Xc))) return s;
    k_copy_cols<<<cdiv(nn * ncols, 256), 256, 0, c->stream>>>(nn, ncols, XC, ldx, Xc, ldd);
    Xd = Xc;
  }
  const int nx = c->nf + (c->nproj ? 1 : 0);
  const int64_t nq = (int64_t)c->natoms * nx;      // coefficient rows
  const int64_t ldq = (ncols + 1) & ~1;            // own buffers: pairs are aligned
  const CoupleSet &cE = c->cpl_e, &cK = c->cpl_k;
  const int64_t prow = c->nf > 0 ? (int64_t)c->nf * cE.n_boxpairs : 0;
  double *Q = nullptr, *R = nullptr, *Yp = nullptr;
  if (nq) {
    if ((s = efe_ws(c, 1, (size_t)(nq + c->nproj) * ldq * 8, (void **)&Q))) return s;
    if ((s = efe_ws(c, 11, (size_t)std::max<int64_t>(c->n_enr, 1) * ldq * 8, (void **)&R)))
      return s;
    if ((s = efe_ws(c, 9, (size_t)std::max<int64_t>(prow + cK.n_boxpairs, 1) * ncols * 8,
                    (void **)&Yp)))
      return s;
  }
  const EpiArgs ec{ep.alpha, ep.beta, ep.gamma, ep.Z1, ep.Z2, ep.G, ep.Cl};
  const bool f32 = prec == EFE_FP32;
  const int t_cls = ncols <= 16 ? EFE_T_APPLY_NARROW : EFE_T_APPLY;
  const int t_apply = efe_timer_begin(c, t_cls);
  // 1. cell Hamiltonians by tensor products, into a workspace that the node
  //    update sums (one launch, fixed order); without room for it, added to
  //    Y^C colour by colour below
  //    (rows of whole 64-byte pieces where there is room: 37 vectors on 4,096
  //    cells 346 us, 451 with pieces of neighbouring rows in one)
  int64_t ldc = ncols <= 16 ? ncols : (ncols + 7) & ~7;
  double *Yc = tp ? efe_ws_try(c, (size_t)c->n_cells * c->nloc * ldc * 8) : nullptr;
  if (tp && !Yc && ldc > ldq) {
    ldc = ldq;
    Yc = efe_ws_try(c, (size_t)c->n_cells * c->nloc * ldc * 8);
  }
  if (Yc && (s = efe_tp_apply(c, XC, ldx, minv, ncols, Yc, ldc, nullptr, 0, 0.0))) return s;
  // 2. coefficients: [E ; P^C] s X^C by boxes, their sums, the dense part (Y^E
  //    and the projector coefficients W)
  if (nq) {
    const int t = efe_timer_begin(c, EFE_T_POST);
    GatherArgs<double> g{};
    g.X = XC;
    g.minv = c->d_minv;
    g.ldx = ldx;
    g.ldp = ncols;
    g.prow = prow;
    g.Yp = Yp;
    g.E = box_set<double>(cE, false, cE.d_T2);
    g.K = box_set<double>(cK, false, cK.d_T2);
    g.g = node_grid(c);
    g.ncols = ncols;
    g.scaled = minv;
    g.vec = xvec;
    if (f32) {
      GatherArgs<float> h{};
      h.items = c->d_items[0];
      h.X = g.X;
      h.minv = g.minv;
      h.ldx = g.ldx;
      h.ldp = g.ldp;
      h.prow = g.prow;
      h.Yp = g.Yp;
      h.E = box_set<float>(cE, false, cE.d_T2f);
      h.K = g.K;
      h.g = g.g;
      h.ncols = ncols;
      h.scaled = g.scaled;
      h.vec = g.vec;
      h.nre = cE.n_rb;
      launch_box_gather(c, h, c->n_items[0]);
    }
    g.items = c->d_items[f32 ? 1 : 2];
    g.nre = f32 ? 0 : cE.n_rb;
    g.nrk = cK.n_rb;
    launch_box_gather(c, g, c->n_items[f32 ? 1 : 2]);
    SumArgs sa{cE.d_at_ptr, cE.d_at_pos, cK.d_at_ptr, cK.d_at_pos, Yp, XE, minv ? c->d_Mee_inv : nullptr,
               ncols, lde, ldq, prow, Q, R, c->nf, nx, ncols, c->nf ? nullptr : c->d_D, Q + nq * ldq};
    if (ncols <= 16) {
      int cw = 1;
      while (cw < ncols) cw *= 2;
      k_coef_sum_narrow<<<c->natoms, 64 * nx, 0, c->stream>>>(sa, cw);
    } else {
      k_coef_sum<<<dim3(c->natoms, cdiv(ncols, 64)), 64 * nx, 0, c->stream>>>(sa);
    }
    EpiArgs ee = ec;
    if (ee.Z1) ee.Z1 += nn * ldy;
    if (ee.Z2) ee.Z2 += nn * ldy;
    if (ee.G) ee.G += nn * ldy;
    if (c->nf > 0 && ncols <= 16)
      k_coef_dense<1><<<dim3(cdiv(nq, 16), 1), 256, 0, c->stream>>>(nq, c->nf, nx, ncols, c->d_S, Q,
                                                                   ldq, R, ee, Y + nn * ldy, ldy);
    else if (c->nf > 0)
      k_coef_dense<5><<<dim3(cdiv(nq, 16), cdiv(ncols, 80)), 256, 0, c->stream>>>(
          nq, c->nf, nx, ncols, c->d_S, Q, ldq, R, ee, Y + nn * ldy, ldy);
    efe_timer_end(c, EFE_T_POST, t);
  }
  // 3. every other term of Y^C
  {
    const int t = efe_timer_begin(c, EFE_T_PRE);
    const bool vec = ldy % 2 == 0 && al(Y) && al(ep.Z1) && al(ep.Z2) && al(ep.G);
    if (f32) {
      NodeArgs<float> a{{}, {}, Q, Yc, ldq, ldc, nq, nx, ncols, 1, node_grid(c), ec, Y, ldy, vec};
      launch_node_update(c, a, (const float *)cE.d_T1f);
    } else {
      NodeArgs<double> a{{}, {}, Q, Yc, ldq, ldc, nq, nx, ncols, 1, node_grid(c), ec, Y, ldy, vec};
      launch_node_update(c, a, (const double *)cE.d_T1);
    }
    efe_timer_end(c, EFE_T_PRE, t);
  }
  // 4. cell products that are added to Y^C colour by colour
  if (tp) {
    if (!Yc && (s = efe_tp_apply(c, XC, ldx, minv, ncols, nullptr, 0, Y, ldy, ep.alpha))) return s;
  } else if (prec == EFE_FP64 && ncols <= 16) {
    launch_cell3<double, 6, 1>(c, c->d_Htile64, Xd, ldd, scale, Y, ldy, ep.alpha, ncols);
  } else if (prec == EFE_FP64) {
    launch_cell3<double, 1, 10>(c, c->d_Htile64, Xd, ldd, scale, Y, ldy, ep.alpha, ncols);
  } else if (f32 && ncols <= 16) {
    launch_cell3<float, 6, 1>(c, c->d_Htile32, Xd, ldd, scale, Y, ldy, ep.alpha, ncols);
  } else if (f32) {
    launch_cell3<float, 2, 10>(c, c->d_Htile32, Xd, ldd, scale, Y, ldy, ep.alpha, ncols);
  } else {
    const int NT = 32;
    const int ntiles = (int)cdiv(ncols, NT);
    const size_t shm = (size_t)NT * (c->KS32 * 32 + 8) * 2;
    for (int col = 0; col < 8; ++col) {
      const int nc = c->colour_offsets[col + 1] - c->colour_offsets[col];
      if (nc == 0) continue;
      const int64_t nblk = cdiv(nc, 8) * 8 * ntiles;
      const int t = efe_timer_begin(c, EFE_T_CELL);
      k_cell_bf16<32><<<nblk, 256, shm, c->stream>>>(
          nc, ntiles, c->d_colour_order + c->colour_offsets[col], c->d_c2g, c->nloc, c->RB,
          c->KS32, (const v8bf *)c->d_Htile16, Xd, ldd, scale, Y, ldy, c->d_minv, ncols,
          ep.alpha);
      efe_timer_end(c, EFE_T_CELL, t);
    }
  }
  efe_timer_end(c, t_cls, t_apply);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}

efe_status efe_transform_cfe(efe_ctx *c, const double *X, int64_t ldx, double *Xh, int64_t ldh,
                             int ncols) {
  if (ncols <= 0) return EFE_OK;
  k_pre<<<cdiv(c->n_nodes, 32), 256, 0, c->stream>>>(c->n_nodes, ncols, X, ldx, c->d_minv,
                                                     X + c->n_nodes * ldx, ldx, c->d_g_ptr,
                                                     c->d_g_atom, c->d_Cg, c->nf, Xh, ldh);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}

efe_status efe_apply_M_internal(efe_ctx *c, const double *X, int64_t ldx, double *Y, int64_t ldy,
                                int ncols) {
  if (ncols <= 0) return EFE_OK;
  k_rowscale<<<cdiv(c->n_nodes * ncols, 256), 256, 0, c->stream>>>(c->n_nodes, ncols, c->d_m_int,
                                                                   X, ldx, Y, ldy);
  HIPCHK(c, hipGetLastError());
  if (c->n_enr)
    return efe_dgemm(c, false, false, c->n_enr, ncols, c->n_enr, 1.0, c->d_Mee, c->n_enr,
                    X + c->n_nodes * ldx, ldx, 0.0, Y + c->n_nodes * ldy, ldy);
  return EFE_OK;
}

efe_status efe_enr_block_inv(efe_ctx *c, const double *XE, int64_t ldx, double *YE, int64_t ldy,
                             int ncols) {
  if (!c->n_enr || ncols <= 0) return EFE_OK;
  const int64_t n = c->n_enr * ncols;
  k_enr_block_apply<<<cdiv(n, 256), 256, 0, c->stream>>>(c->natoms, c->nf, ncols, c->d_Mee_inv, XE,
                                                         ldx, YE, ldy);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}

efe_status efe_apply_Minv_internal(efe_ctx *c, const double *X, int64_t ldx, double *Y,
                                   int64_t ldy, int ncols) {
  if (ncols <= 0) return EFE_OK;
  k_rowscale<<<cdiv(c->n_nodes * ncols, 256), 256, 0, c->stream>>>(c->n_nodes, ncols, c->d_minv, X,
                                                                   ldx, Y, ldy);
  HIPCHK(c, hipGetLastError());
  return efe_enr_block_inv(c, X + c->n_nodes * ldx, ldx, Y + c->n_nodes * ldy, ldy, ncols);
}

// ------------------------------------------------------------------ C ABI
static efe_status check_block(efe_ctx *c, const void *X, const void *Y, int ncols, int64_t ld) {
  if (!c) return EFE_EINVAL;
  if (!X || !Y || ncols < 0 || ld < ncols || ld < 1) EFE_FAIL(c, EFE_EINVAL, "bad block arguments");
  if (X == Y) EFE_FAIL(c, EFE_EINVAL, "input and output blocks must differ");
  return EFE_OK;
}

extern "C" efe_status efe_local_potential(efe_ctx *c, double *vq) {
  if (!c) return EFE_EINVAL;
  if (!vq) EFE_FAIL(c, EFE_EINVAL, "null vq");
  return efe_launch_local_potential(c, vq);
}

extern "C" efe_status efe_set_potential(efe_ctx *c, const double *vq, int32_t precisions) {
  if (!c) return EFE_EINVAL;
  if (!vq) EFE_FAIL(c, EFE_EINVAL, "null vq");
  if (precisions & ~((1 << EFE_FP32) | (1 << EFE_BF16))) EFE_FAIL(c, EFE_EINVAL, "bad precision mask");
  return efe_build_operators(c, vq, precisions);
}

// wide blocks go through the apply in column chunks of the widest register
// tile, so its workspaces stay n_nodes x 160
static efe_status apply_H_chunked(efe_ctx *c, const double *X, double *Y, int32_t ncols,
                                  int64_t ld, int prec) {
  efe_status s;
  for (int32_t j0 = 0; j0 < ncols; j0 += EFE_COL_CHUNK) {
    const int32_t nc = std::min<int32_t>(EFE_COL_CHUNK, ncols - j0);
    if ((s = efe_apply_H_internal(c, X + j0, ld, false, X + c->n_nodes * ld + j0, ld, Y + j0, ld,
                                  nc, prec)))
      return s;
  }
  return EFE_OK;
}

extern "C" efe_status efe_apply_H(efe_ctx *c, const double *X, double *Y, int32_t ncols,
                                  int64_t ld) {
  efe_status s = check_block(c, X, Y, ncols, ld);
  if (s) return s;
  return apply_H_chunked(c, X, Y, ncols, ld, EFE_FP64);
}

extern "C" efe_status efe_apply_H_prec(efe_ctx *c, const double *X, double *Y, int32_t ncols,
                                       int64_t ld, int32_t prec) {
  efe_status s = check_block(c, X, Y, ncols, ld);
  if (s) return s;
  if (prec != EFE_FP64 && prec != EFE_FP32 && prec != EFE_BF16)
    EFE_FAIL(c, EFE_EINVAL, "bad precision");
  return apply_H_chunked(c, X, Y, ncols, ld, prec);
}

extern "C" efe_status efe_apply_M(efe_ctx *c, const double *X, double *Y, int32_t ncols,
                                  int64_t ld) {
  efe_status s = check_block(c, X, Y, ncols, ld);
  if (s) return s;
  return efe_apply_M_internal(c, X, ld, Y, ld, ncols);
}

extern "C" efe_status efe_apply_Minv_approx(efe_ctx *c, const double *X, double *Y, int32_t ncols,
                                            int64_t ld) {
  efe_status s = check_block(c, X, Y, ncols, ld);
  if (s) return s;
  return efe_apply_Minv_internal(c, X, ld, Y, ld, ncols);
}
