// Learned initial density: quadrature export, atom-centred descriptors, the
// density MLP (forward, backward, loss gradient, Adam) and the guess
// ρ_0 = max(ρ_SAD + Δρ, 0) renormalized to the electron count, with the
// superposition of atomic densities as fallback.  All MLP arithmetic is FP32;
// descriptors are formed in FP64 and stored in FP32.
#include <cmath>

#include "efe_device.h"

// positions and weights (reference weight times cell Jacobian) of every
// Gauss point, cell by cell
__global__ void k_quadrature(MeshGeo g, const double *__restrict__ xq1,
                             const double *__restrict__ W3, double *__restrict__ xq,
                             double *__restrict__ wq) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t nq = (int64_t)g.ncell[0] * g.ncell[1] * g.ncell[2] * g.nqp;
  if (idx >= nq) return;
  const int q = (int)(idx % g.nqp);
  if (xq) {
    double x[3];
    quad_point(g, xq1, (int)(idx / g.nqp), q, x);
    xq[3 * idx] = x[0];
    xq[3 * idx + 1] = x[1];
    xq[3 * idx + 2] = x[2];
  }
  if (wq) wq[idx] = W3[q];
}

extern "C" efe_status efe_get_quadrature(efe_ctx *c, double *xq, double *wq) {
  if (!c) return EFE_EINVAL;
  if (!xq && !wq) EFE_FAIL(c, EFE_EINVAL, "both outputs null");
  const MeshGeo g = mesh_geo(c);
  k_quadrature<<<cdiv(c->n_qpts, 256), 256, 0, c->stream>>>(g, c->d_xq1, c->d_W3, xq, wq);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}

// ------------------------------------------------------------------ descriptors
namespace {
constexpr int KNEAR = 16;   // nearest atoms per point
constexpr int NRAD = 8;     // radial Gaussians exp(-(d - n)^2 / 2), n = 0..7
constexpr int MLP_IN = 25;  // 8 x 3 power-spectrum entries + log rho_SAD
constexpr int MLP_H = 128;
// flat parameter layout: W1 [128][25], b1, W2 [128][128], b2, W3, b3, W4 [128], b4
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + MLP_H * MLP_IN, OFF_W2 = OFF_B1 + MLP_H,
              OFF_B2 = OFF_W2 + MLP_H * MLP_H, OFF_W3 = OFF_B2 + MLP_H,
              OFF_B3 = OFF_W3 + MLP_H * MLP_H, OFF_W4 = OFF_B3 + MLP_H, OFF_B4 = OFF_W4 + MLP_H,
              N_PARAMS = OFF_B4 + 1;
constexpr double RHO_FLOOR = 1e-12;
constexpr int TP = 64;      // points per work-group tile of the MLP kernels
}  // namespace

__device__ inline double dist2_nofma(double x0, double x1, double x2, const double *a) {
#pragma clang fp contract(off)
  const double dx = x0 - a[0], dy = x1 - a[1], dz = x2 - a[2];
  return (dx * dx + dy * dy) + dz * dz;
}

// One thread per point: the 16 nearest atoms (ties by lower index, kept in
// registers by an unrolled insertion), then for every radial Gaussian n the
// sums A_lm = sum_I g_n(d_I) Y_lm(u_I) and the power spectrum per l.
__global__ __launch_bounds__(256) void k_descriptors(int64_t npts, const double *__restrict__ pts,
                                                     int natoms, const double *__restrict__ xyz,
                                                     const double *__restrict__ rho_sad,
                                                     const float *__restrict__ shift,
                                                     const float *__restrict__ scale,
                                                     float *__restrict__ feat) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= npts) return;
  const double x0 = pts[3 * p], x1 = pts[3 * p + 1], x2 = pts[3 * p + 2];
  double kd[KNEAR];
  int ki[KNEAR];
#pragma unroll
  for (int j = 0; j < KNEAR; ++j) {
    kd[j] = INFINITY;
    ki[j] = -1;
  }
  for (int I = 0; I < natoms; ++I) {
    const double d2 = dist2_nofma(x0, x1, x2, xyz + 3 * I);
    if (d2 < kd[KNEAR - 1]) {
#pragma unroll
      for (int j = KNEAR - 1; j > 0; --j) {
        const bool up = kd[j - 1] > d2;
        const bool here = !up && kd[j] > d2;
        kd[j] = up ? kd[j - 1] : (here ? d2 : kd[j]);
        ki[j] = up ? ki[j - 1] : (here ? I : ki[j]);
      }
      if (kd[0] > d2) {
        kd[0] = d2;
        ki[0] = I;
      }
    }
  }
  const double c0 = 0.5 / sqrt(M_PI), c1 = sqrt(3.0 / (4.0 * M_PI)), c2 = 0.5 * sqrt(15.0 / M_PI),
               c20 = 0.25 * sqrt(5.0 / M_PI), c22 = 0.25 * sqrt(15.0 / M_PI);
  float *f = feat + p * MLP_IN;
  for (int n = 0; n < NRAD; ++n) {
    double A[9];
#pragma unroll
    for (int m = 0; m < 9; ++m) A[m] = 0.0;
#pragma unroll
    for (int j = 0; j < KNEAR; ++j) {
      if (ki[j] >= 0) {
        const double *a = xyz + 3 * ki[j];
        const double vx = x0 - a[0], vy = x1 - a[1], vz = x2 - a[2];
        const double d = sqrt(kd[j]);
        const double g = exp(-0.5 * (d - n) * (d - n));
        A[0] += g * c0;
        if (d > 0.0) {
          const double ux = vx / d, uy = vy / d, uz = vz / d;
          A[1] += g * c1 * uy;
          A[2] += g * c1 * uz;
          A[3] += g * c1 * ux;
          A[4] += g * c2 * ux * uy;
          A[5] += g * c2 * uy * uz;
          A[6] += g * c20 * (3.0 * uz * uz - 1.0);
          A[7] += g * c2 * ux * uz;
          A[8] += g * c22 * (ux * ux - uy * uy);
        }
      }
    }
    const double P[3] = {A[0] * A[0], A[1] * A[1] + A[2] * A[2] + A[3] * A[3],
                         A[4] * A[4] + A[5] * A[5] + A[6] * A[6] + A[7] * A[7] + A[8] * A[8]};
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      const int i = 3 * n + l;
      f[i] = shift ? (float)((P[l] - (double)shift[i]) / (double)scale[i]) : (float)P[l];
    }
  }
  const double lr = log(fmax(rho_sad[p], RHO_FLOOR));
  f[24] = shift ? (float)((lr - (double)shift[24]) / (double)scale[24]) : (float)lr;
}

// ------------------------------------------------------------------ MLP
__device__ inline float sigm(float z) { return 1.0f / (1.0f + __expf(-z)); }

// The layers run on v_mfma_f32_16x16x4 with neurons as rows and points as
// columns, a wave per 16 neurons.  A wave's weights
// stay in its registers for the whole launch and the work-groups loop over
// 64-point tiles, so the only traffic is a tile's activations through LDS; the
// scalar products this replaces ran at 20 TFLOP/s (forward) and staged 64 KB of
// weights per tile and layer.  65,536 points: forward 68 us (before 241), the
// backward layers 73, 68 and 20 us (329, 329 and 241), where the matrix cores
// alone would take 32, 29, 29 and 4 us; the activations and their exponentials
// are the rest.  v_mfma_f32_16x16x4 adds its four products one after the other
// as fused multiply-adds, so sums taken in the order of k are those of a scalar
// loop, bit for bit.  Two work-groups a CU (forward) need the weights in 128
// registers; at 256 a group had the CU to itself and took 105 us.
typedef float v4m __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4m mfma4(float a, float b, v4m c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// LDS row strides of [neuron][point] tiles.  Backward: 16 neurons x 4 points (a
// gradient's operand) and, with the contraction index in the order kidx, 4
// neurons x 16 points (the other operand) hit 64 different banks; forward: the
// same for 4 consecutive neurons x 16 points.
constexpr int BS = TP + 4, FS = TP + 16;
__device__ __forceinline__ int kidx(int s, int lk) { return 16 * (s / 4) + 4 * lk + s % 4; }

// A scalar base pointer: left alone, each of a loop's addresses becomes a running
// 64-bit pointer in vector registers, which the weights need.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T *uniform(T *p) {
  auto *g = (__attribute__((address_space(1))) T *)p;
  asm volatile("" : "+s"(g));
  return g;
}

// Forward pass of 64-point tiles, one layer after the other.  acts (optional)
// receives the pre-activations z1..z3.  Wave w holds the weights of neurons
// 16 w ..; a layer's output replaces its input in LDS.
template <int K>
__device__ __forceinline__ void fwd_weights(const float *__restrict__ W, int n, int lk,
                                            float (&w)[(K + 3) / 4]) {
#pragma unroll
  for (int s = 0; s < (K + 3) / 4; ++s) {
    const int k = 4 * s + lk;
    const float x = W[n * K + min(k, K - 1)];
    w[s] = k < K ? x : 0.0f;
  }
}

// the same for K = 128 from consecutive loads, transposed through the wave's part
// of H (64 scattered loads took 10 us longer)
__device__ __forceinline__ void fwd_weights_h(const float *__restrict__ W, float *H, int wave,
                                              int li, int lk, float (&w)[MLP_H / 4]) {
  float *A = H + wave * 16 * BS;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int r = 0; r < 16; r += 4)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        A[(r + lk) * BS + 4 * li + i] = W[(16 * wave + r + lk) * MLP_H + 64 * h + 4 * li + i];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 16; ++s) w[16 * h + s] = A[li * BS + 4 * s + lk];
    __syncthreads();
  }
}

// z (neurons n0 + 4 lk + v, points 16 c + li) = W h + b, the products of a sum
// in the order of k.  H is [neuron k][point] with row stride FS; SWZ: 16-point
// blocks permuted by hcol, so that the rows 4 lk + v that a layer's output
// stores together lie in different banks, as the rows 4 s + lk read here do.
__device__ __forceinline__ int hcol(int c, int row4) { return 16 * (c ^ (row4 & 3)); }
template <int K, bool SWZ>
__device__ __forceinline__ void fwd_layer(const float (&w)[(K + 3) / 4], const float *b,
                                          const float *H, int li, int lk, v4m (&z)[4]) {
#pragma unroll
  for (int c = 0; c < 4; ++c) z[c] = *(const v4m *)b;
  int o = lk * FS + li;
  asm volatile("" : "+v"(o));   // row addresses formed here, not kept
#pragma unroll
  for (int s = 0; s < (K + 3) / 4; ++s) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      z[c] = mfma4(w[s], H[o + 4 * s * FS + (SWZ ? hcol(c, s) : 16 * c)], z[c]);
    // keeps the LDS reads near their use: hoisted, they push the weights to scratch
    if (s % 2 == 1) __builtin_amdgcn_sched_barrier(0);
  }
}

__global__ __launch_bounds__(512, 4) void k_mlp_fwd(int64_t npts, const float *__restrict__ prm,
                                                    const float *__restrict__ X,
                                                    float *__restrict__ y,
                                                    float *__restrict__ acts) {
  constexpr int KX = 32, NX = TP * KX / 512;   // padded inputs, those a thread brings
  __shared__ float Hx[KX * FS];
  __shared__ float H[MLP_H * FS];
  __shared__ __align__(16) float bs[4][MLP_H];          // b1, b2, b3, w4
  const int t = threadIdx.x, wave = t / 64, lane = t % 64, li = lane % 16, lk = lane / 16;
  const int n0 = 16 * wave + 4 * lk;
  float w1[7], w2[32], w3[32];
  fwd_weights<MLP_IN>(prm + OFF_W1, 16 * wave + li, lk, w1);
  fwd_weights_h(prm + OFF_W2, H, wave, li, lk, w2);
  fwd_weights_h(prm + OFF_W3, H, wave, li, lk, w3);
  if (t < MLP_H) {
    bs[0][t] = prm[OFF_B1 + t];
    bs[1][t] = prm[OFF_B2 + t];
    bs[2][t] = prm[OFF_B3 + t];
    bs[3][t] = prm[OFF_W4 + t];
  }
  const int64_t ntiles = (npts + TP - 1) / TP;
  float xr[NX];
  auto load = [&](int64_t tile) {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int e = t + 512 * i;
      auto *a = uniform(X + tile * TP * MLP_IN);
      const int last = (int)min<int64_t>(TP, npts - tile * TP) - 1;
      xr[i] = a[(unsigned)(min(e / KX, last) * MLP_IN + min(e % KX, MLP_IN - 1))];
    }
  };
  load(min((int64_t)blockIdx.x, ntiles - 1));
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t p0 = tile * TP;
    const int np = (int)min<int64_t>(TP, npts - p0);
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int e = t + 512 * i, p = e / KX, k = e % KX;
      Hx[k * FS + p] = p < np && k < MLP_IN ? xr[i] : 0.0f;
    }
    __syncthreads();
    load(min(tile + (int64_t)gridDim.x, ntiles - 1));
    v4m z[4];
    auto finish = [&](int l) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int p = 16 * c + li;
        if (acts) {
          auto *a = uniform(acts + ((int64_t)l * npts + p0 + 16 * c) * MLP_H);
          if (p < np) *(__attribute__((address_space(1))) v4m *)&a[(unsigned)(li * MLP_H + n0)] = z[c];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) z[c][v] *= sigm(z[c][v]);
        int o = n0 * FS + hcol(c, lk) + li;
        asm volatile("" : "+v"(o));   // formed here, not kept
#pragma unroll
        for (int v = 0; v < 4; ++v) H[o + v * FS] = z[c][v];
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    fwd_layer<MLP_IN, false>(w1, &bs[0][n0], Hx, li, lk, z);
    finish(0);
    __syncthreads();
    fwd_layer<MLP_H, true>(w2, &bs[1][n0], H, li, lk, z);
    __syncthreads();
    finish(1);
    __syncthreads();
    fwd_layer<MLP_H, true>(w3, &bs[2][n0], H, li, lk, z);
    __syncthreads();
    finish(2);
    __syncthreads();
    // output layer, a wave's 16 points: one row of a product
    if (wave < TP / 16) {
      v4m o = {prm[OFF_B4], 0.f, 0.f, 0.f};
      const float on = li == 0 ? 1.0f : 0.0f;
#pragma unroll 8
      for (int s = 0; s < MLP_H / 4; ++s)
        o = mfma4(on * bs[3][4 * s + lk], H[(4 * s + lk) * FS + hcol(wave, s) + li], o);
      const int p = 16 * wave + li;
      if (lk == 0 && p < np) y[p0 + p] = o[0];
    }
  }
}

// Backward of one hidden layer z = W h + b, h = silu(z_prev) (KIN = 128) or the
// standardized input (KIN = 25), over 64-point tiles: gW += dz^T h and gb += sum
// dz in registers, added to grads once per work-group; dz_prev = (dz W)
// silu'(z_prev) for KIN = 128.  HEAD: dz = dy W4 silu'(z) is formed here from z
// (the last layer's), with gW4 += dy silu(z) and gb4 += dy.  Eight waves, wave w
// on neurons 16 w ..: their dz and h on the way into LDS, rows of gW, and rows of
// dz_prev with W^T in registers.  A thread's tile values are those of its
// dz_prev, so silu'(z_prev) never leaves its registers.  The tiles alternate
// between two LDS buffers with one barrier a tile, so one wave's products run
// beside another's activations, and the next tile's loads beside both.
template <int KIN, bool HEAD>
__global__ __launch_bounds__(512) void k_mlp_bwd_layer(int64_t npts, const float *__restrict__ prm,
                                                       int offW, int offB,
                                                       const float *__restrict__ dzin,
                                                       const float *__restrict__ dy,
                                                       const float *__restrict__ hin,
                                                       float *__restrict__ dzprev,
                                                       float *__restrict__ grads) {
  constexpr bool PREV = KIN == MLP_H;
  constexpr int KB = (KIN + 15) / 16;          // 16-column blocks of gW
  constexpr int KE = PREV ? 0 : TP * 32 / 512; // inputs a thread brings
  extern __shared__ float sm[];
  constexpr int NB = (MLP_H + 16 * KB) * BS;   // dz [neuron][point], h [input][point]
  const int t = threadIdx.x, wave = t / 64, lane = t % 64, li = lane % 16, lk = lane / 16;
  const int n0 = 16 * wave + 4 * lk;           // this thread's neurons, at points 16 c + li
  float wt[PREV ? 32 : 1];                     // W^T: rows 16 wave + li, columns kidx
  if constexpr (PREV)
#pragma unroll
    for (int s = 0; s < 32; ++s) wt[s] = prm[offW + kidx(s, lk) * MLP_H + 16 * wave + li];
  v4m gw[KB];
#pragma unroll
  for (int c = 0; c < KB; ++c) gw[c] = (v4m){0.f, 0.f, 0.f, 0.f};
  v4m gb = {0.f, 0.f, 0.f, 0.f}, g4 = gb, w4 = gb;
  float gb4 = 0.0f;
  if constexpr (HEAD)
#pragma unroll
    for (int v = 0; v < 4; ++v) w4[v] = prm[OFF_W4 + n0 + v];
  v4m dr[4], hr[PREV ? 4 : 1];
  float yr[HEAD ? 4 : 1], xr[PREV ? 1 : KE];
  const int64_t ntiles = (npts + TP - 1) / TP;
  auto load = [&](int64_t tile) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int64_t p = min(tile * TP + 16 * c + li, npts - 1);
      dr[c] = *(const v4m *)&dzin[p * MLP_H + n0];
      if constexpr (HEAD) yr[c] = dy[p];
      if constexpr (PREV) hr[c] = *(const v4m *)&hin[p * MLP_H + n0];
    }
#pragma unroll
    for (int i = 0; i < KE; ++i) {
      const int e = t + 512 * i;
      xr[i] = hin[min(tile * TP + e / 32, npts - 1) * KIN + min(e % 32, KIN - 1)];
    }
  };
  load(blockIdx.x);
  int par = 0;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x, par ^= 1) {
    const int64_t p0 = tile * TP;
    const int np = (int)min<int64_t>(TP, npts - p0);
    float *D = sm + par * NB, *H = D + MLP_H * BS;
    v4m sp[PREV ? 4 : 1];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int p = 16 * c + li;
      const bool on = p < np;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float d = on ? dr[c][v] : 0.0f;
        if constexpr (HEAD) {
          const float s = sigm(d), u = on ? yr[c] : 0.0f;
          g4[v] = fmaf(u, d * s, g4[v]);
          d = u * w4[v] * (s * (1.0f + d * (1.0f - s)));
        }
        gb[v] += d;
        D[(n0 + v) * BS + p] = d;
        if constexpr (PREV) {
          const float z = on ? hr[c][v] : 0.0f, s = sigm(z);
          H[(n0 + v) * BS + p] = z * s;
          sp[c][v] = s * (1.0f + z * (1.0f - s));
        }
      }
      if constexpr (HEAD) gb4 += on ? yr[c] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < KE; ++i) {
      const int e = t + 512 * i, p = e / 32, k = e % 32;
      H[k * BS + p] = p < np && k < KIN ? xr[i] : 0.0f;
    }
    __syncthreads();
    load(min(tile + (int64_t)gridDim.x, ntiles - 1));
    if constexpr (PREV) {
      v4m acc[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = (v4m){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 32; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          acc[c] = mfma4(wt[s], D[kidx(s, lk) * BS + 16 * c + li], acc[c]);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int p = 16 * c + li;
        if (p < np) *(v4m *)&dzprev[(p0 + p) * MLP_H + n0] = acc[c] * sp[c];
      }
    }
    // gW rows 16 wave .., columns 16 c ..: the sum over the points
#pragma unroll 4
    for (int s = 0; s < TP / 4; ++s) {
      const float a = D[(16 * wave + li) * BS + 4 * s + lk];
#pragma unroll
      for (int c = 0; c < KB; ++c) gw[c] = mfma4(a, H[(16 * c + li) * BS + 4 * s + lk], gw[c]);
    }
  }
  __syncthreads();
  // through LDS, so that a wave's atomics hit consecutive addresses and the
  // work-groups, which end together, start at different ones
#pragma unroll
  for (int c = 0; c < KB; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int k = 16 * c + li;
      if (k < KIN) sm[(n0 + v) * KIN + k] = gw[c][v];
    }
  float *ge = sm + MLP_H * KIN;
#pragma unroll
  for (int o = 1; o < 16; o *= 2) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      gb[v] += __shfl_xor(gb[v], o);
      if (HEAD) g4[v] += __shfl_xor(g4[v], o);
    }
    if (HEAD) gb4 += __shfl_xor(gb4, o);
  }
  if (li == 0)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      ge[n0 + v] = gb[v];
      if (HEAD) ge[MLP_H + n0 + v] = g4[v];
    }
  if (HEAD && t == 0) ge[2 * MLP_H] = gb4;
  __syncthreads();
  constexpr int NW = MLP_H * KIN;
  int i = (int)((int64_t)blockIdx.x * NW / gridDim.x) + t;
  for (int e = t; e < NW; e += 512, i += 512) {
    if (i >= NW) i -= NW;
    atomicAdd(&grads[offW + i], sm[i]);
  }
  if (t < MLP_H) atomicAdd(&grads[offB + t], ge[t]);
  if (HEAD && t <= MLP_H) atomicAdd(&grads[OFF_W4 + t], ge[MLP_H + t]);   // b4 follows W4
}

// sums[0] += sum w, sums[1] += sum w (y - t)^2 (FP64)
__global__ __launch_bounds__(256) void k_loss_sums(int64_t n, const float *__restrict__ y,
                                                   const float *__restrict__ tg,
                                                   const float *__restrict__ w,
                                                   double *__restrict__ sums) {
  __shared__ double s0[256], s1[256];
  double a = 0.0, b = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double r = (double)y[i] - (double)tg[i];
    a += w[i];
    b += w[i] * r * r;
  }
  s0[threadIdx.x] = a;
  s1[threadIdx.x] = b;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      s0[threadIdx.x] += s0[threadIdx.x + s];
      s1[threadIdx.x] += s1[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    atomicAdd(&sums[0], s0[0]);
    atomicAdd(&sums[1], s1[0]);
  }
}

__global__ void k_loss_grad(int64_t n, const float *__restrict__ y, const float *__restrict__ tg,
                            const float *__restrict__ w, const double *__restrict__ sums,
                            float *__restrict__ dy) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) dy[i] = (float)(2.0 * (double)w[i] * ((double)y[i] - (double)tg[i]) / sums[0]);
}

__global__ void k_fill_f32(int64_t n, float *__restrict__ x, float v) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) x[i] = v;
}

__global__ void k_fill_f64(int64_t n, double *__restrict__ x, double v) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) x[i] = v;
}

__global__ void k_adam(int64_t n, float *__restrict__ prm, const float *__restrict__ g,
                       float *__restrict__ m, float *__restrict__ v, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  prm[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// rho0 = max(rho_SAD + s_t y, 0); sums[0] += int rho0, sums[1] counts non-finite values
__global__ __launch_bounds__(256) void k_guess(int64_t n, const double *__restrict__ sad,
                                               const float *__restrict__ y, double st,
                                               const double *__restrict__ wq,
                                               double *__restrict__ rho,
                                               double *__restrict__ sums) {
  __shared__ double s0[256], s1[256];
  double a = 0.0, b = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double r = sad[i] + st * (double)y[i];
    if (!isfinite(r)) {
      b += 1.0;
      rho[i] = 0.0;
    } else {
      const double c = fmax(r, 0.0);
      rho[i] = c;
      a += wq[i] * c;
    }
  }
  s0[threadIdx.x] = a;
  s1[threadIdx.x] = b;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      s0[threadIdx.x] += s0[threadIdx.x + s];
      s1[threadIdx.x] += s1[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    atomicAdd(&sums[0], s0[0]);
    atomicAdd(&sums[1], s1[0]);
  }
}

__global__ void k_scale_f64(int64_t n, double *__restrict__ x, double f) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) x[i] *= f;
}

// ------------------------------------------------------------------ C ABI
namespace {
efe_status gfail(efe_status code, const std::string &msg) {
  efe_set_global_error(msg);
  return code;
}
#define GCHK(call)                                                                   \
  do {                                                                               \
    hipError_t e_ = (call);                                                          \
    if (e_ != hipSuccess)                                                            \
      return gfail(EFE_EHIP, std::string(#call) + " failed: " + hipGetErrorString(e_)); \
  } while (0)

constexpr size_t BWD_LDS_128 = 2 * (size_t)(2 * MLP_H * BS) * sizeof(float);
constexpr size_t BWD_LDS_25 = 2 * (size_t)((MLP_H + 32) * BS) * sizeof(float);

efe_status lds_attrs() {
  static bool done = false;
  if (done) return EFE_OK;
  const void *big[] = {(const void *)k_mlp_bwd_layer<MLP_H, true>,
                       (const void *)k_mlp_bwd_layer<MLP_H, false>,
                       (const void *)k_mlp_bwd_layer<MLP_IN, false>};
  for (const void *f : big)
    GCHK(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)BWD_LDS_128));
  done = true;
  return EFE_OK;
}

efe_status mlp_forward(hipStream_t s, const float *prm, const float *feat, int64_t npts, float *out,
                       float *acts) {
  if (npts == 0) return EFE_OK;
  // two work-groups a CU
  k_mlp_fwd<<<(int)std::min<int64_t>(cdiv(npts, TP), 512), 512, 0, s>>>(npts, prm, feat, out, acts);
  GCHK(hipGetLastError());
  return EFE_OK;
}
}  // namespace

extern "C" efe_status efe_descriptors(void *stream, const double *pts, int64_t npts,
                                      const double *xyz, int32_t natoms, const double *rho_sad,
                                      const float *shift, const float *scale, float *feat) {
  if (npts < 0 || natoms < 0 || (npts && (!pts || !rho_sad || !feat)) || (natoms && !xyz) ||
      (!shift) != (!scale))
    return gfail(EFE_EINVAL, "efe_descriptors: bad arguments");
  if (npts == 0) return EFE_OK;
  k_descriptors<<<cdiv(npts, 256), 256, 0, (hipStream_t)stream>>>(npts, pts, natoms, xyz, rho_sad,
                                                                  shift, scale, feat);
  GCHK(hipGetLastError());
  return EFE_OK;
}

extern "C" efe_status efe_mlp_forward(void *stream, const float *params, const float *feat,
                                      int64_t npts, float *out, float *acts) {
  if (npts < 0 || (npts && (!params || !feat || !out)))
    return gfail(EFE_EINVAL, "efe_mlp_forward: bad arguments");
  return mlp_forward((hipStream_t)stream, params, feat, npts, out, acts);
}

extern "C" efe_status efe_mlp_loss_grad(void *stream, const float *out, const float *target,
                                        const float *weight, int64_t npts, float *dout,
                                        double *sums) {
  if (npts <= 0 || !out || !target || !weight || !dout || !sums)
    return gfail(EFE_EINVAL, "efe_mlp_loss_grad: bad arguments");
  hipStream_t s = (hipStream_t)stream;
  k_fill_f64<<<1, 64, 0, s>>>(2, sums, 0.0);
  k_loss_sums<<<(int)std::min<int64_t>(cdiv(npts, 256), 1024), 256, 0, s>>>(npts, out, target,
                                                                            weight, sums);
  k_loss_grad<<<cdiv(npts, 256), 256, 0, s>>>(npts, out, target, weight, sums, dout);
  GCHK(hipGetLastError());
  return EFE_OK;
}

extern "C" efe_status efe_mlp_backward(void *stream, const float *params, const float *feat,
                                       const float *acts, const float *dout, int64_t npts,
                                       float *grads, float *work) {
  if (npts <= 0 || !params || !feat || !acts || !dout || !grads || !work)
    return gfail(EFE_EINVAL, "efe_mlp_backward: bad arguments");
  efe_status st;
  if ((st = lds_attrs())) return st;
  hipStream_t s = (hipStream_t)stream;
  const int64_t zs = npts * MLP_H;
  const float *z1 = acts, *z2 = acts + zs, *z3 = acts + 2 * zs;
  float *A = work, *B = work + zs;
  k_fill_f32<<<cdiv(N_PARAMS, 256), 256, 0, s>>>(N_PARAMS, grads, 0.0f);
  const int gl = (int)std::min<int64_t>(cdiv(npts, TP), 256);
  k_mlp_bwd_layer<MLP_H, true><<<gl, 512, BWD_LDS_128, s>>>(npts, params, OFF_W3, OFF_B3, z3, dout,
                                                           z2, A, grads);
  k_mlp_bwd_layer<MLP_H, false><<<gl, 512, BWD_LDS_128, s>>>(npts, params, OFF_W2, OFF_B2, A, nullptr,
                                                            z1, B, grads);
  k_mlp_bwd_layer<MLP_IN, false><<<gl, 512, BWD_LDS_25, s>>>(npts, params, OFF_W1, OFF_B1, B, nullptr,
                                                            feat, nullptr, grads);
  GCHK(hipGetLastError());
  return EFE_OK;
}

extern "C" efe_status efe_mlp_adam(void *stream, float *params, const float *grads, float *m,
                                   float *v, int64_t n, double lr, double beta1, double beta2,
                                   double eps, int64_t step) {
  if (n <= 0 || !params || !grads || !m || !v || step < 1 || !(lr > 0) || !(beta1 >= 0) ||
      !(beta1 < 1) || !(beta2 >= 0) || !(beta2 < 1) || !(eps > 0))
    return gfail(EFE_EINVAL, "efe_mlp_adam: bad arguments");
  const double c1 = 1.0 / (1.0 - pow(beta1, (double)step));
  const double c2 = 1.0 / (1.0 - pow(beta2, (double)step));
  k_adam<<<cdiv(n, 256), 256, 0, (hipStream_t)stream>>>(n, params, grads, m, v, (float)lr,
                                                        (float)beta1, (float)beta2, (float)eps,
                                                        (float)c1, (float)c2);
  GCHK(hipGetLastError());
  return EFE_OK;
}

extern "C" int64_t efe_mlp_num_params(void) { return N_PARAMS; }

extern "C" efe_status efe_density_guess(efe_ctx *c, const float *params, const float *norm,
                                        int32_t *used_fallback, double *factor) {
  if (!c) return EFE_EINVAL;
  if (!used_fallback || !factor || (params && !norm))
    EFE_FAIL(c, EFE_EINVAL, "efe_density_guess: bad arguments");
  const int64_t nq = c->n_qpts;
  efe_status st;
  double *sad, *rho, *xq, *wq, *sums;
  float *feat, *y, *dnorm;
  if ((st = efe_ws(c, 40, nq * 8, (void **)&sad))) return st;
  if ((st = efe_get_density(c, 2, sad))) return st;
  *used_fallback = 1;
  *factor = 1.0;
  if (!params) return efe_set_density(c, sad);
  if ((st = efe_ws(c, 41, nq * 8, (void **)&rho))) return st;
  if ((st = efe_ws(c, 42, nq * 24, (void **)&xq))) return st;
  if ((st = efe_ws(c, 43, nq * 8, (void **)&wq))) return st;
  if ((st = efe_ws(c, 44, nq * (MLP_IN + 1) * 4, (void **)&feat))) return st;
  if ((st = efe_ws(c, 45, 256, (void **)&sums))) return st;
  if ((st = efe_ws(c, 46, 64 * 4, (void **)&dnorm))) return st;
  y = feat + nq * MLP_IN;
  if ((st = efe_get_quadrature(c, xq, wq))) return st;
  HIPCHK(c, hipMemcpyAsync(dnorm, norm, 2 * MLP_IN * sizeof(float), hipMemcpyHostToDevice,
                           c->stream));
  k_descriptors<<<cdiv(nq, 256), 256, 0, c->stream>>>(nq, xq, c->natoms, c->d_xyz, sad, dnorm,
                                                      dnorm + MLP_IN, feat);
  HIPCHK(c, hipGetLastError());
  if ((st = mlp_forward(c->stream, params, feat, nq, y, nullptr))) {
    c->err = efe_last_error(nullptr);
    return st;
  }
  k_fill_f64<<<1, 64, 0, c->stream>>>(2, sums, 0.0);
  k_guess<<<(int)std::min<int64_t>(cdiv(nq, 256), 2048), 256, 0, c->stream>>>(
      nq, sad, y, (double)norm[2 * MLP_IN], wq, rho, sums);
  HIPCHK(c, hipGetLastError());
  double h[2];
  HIPCHK(c, hipMemcpyAsync(h, sums, 16, hipMemcpyDeviceToHost, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  double n_el = 0.0;
  for (double z : c->Z) n_el += z;
  const double f = h[0] > 0.0 ? n_el / h[0] : INFINITY;
  *factor = f;
  if (h[1] != 0.0 || !std::isfinite(f) || f < 0.9 || f > 1.1) {
    if (h[1] != 0.0) *factor = NAN;
    return efe_set_density(c, sad);
  }
  k_scale_f64<<<cdiv(nq, 256), 256, 0, c->stream>>>(nq, rho, f);
  HIPCHK(c, hipGetLastError());
  *used_fallback = 0;
  return efe_set_density(c, rho);
}
