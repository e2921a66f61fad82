// Coupling of the orthogonalized enrichment and of the projectors to the CFE
// nodes, as dense blocks over boxes of nodes.
//
// The enrichment couples to a node j through E_fj = sum over the cells c of j
// of (B_c - C_c H_c)_fj (Sec. II.B, N^E = phi - C N^C, E = B - C H^cc), formed
// in FP64 per cell and summed over the cells here, so that every node enters
// the products once (per cell, shared faces enter up to eight times: 1.5 times
// the flops at p = 6).  The apply needs E both ways, in two sets of blocks:
//   bricks  4 x 4 x 4 nodes (rows) x the functions of the atoms that touch the
//           brick: Y^C += E^T X^E.  Four 16-row blocks, one a wave; the
//           smaller the brick, the fewer zero entries of E it holds.
//   boxes   8 x 8 x 8 nodes (summation) x those functions (rows): E X^C, one
//           partial row per (box, function).  Larger boxes mean fewer partial
//           rows (0.11 ms of traffic for 64 atoms and 160 vectors, against 0.2
//           with 8 x 8 x 4), at 7% more products.
// The projectors P^C have the same two sets, one function per atom, always in
// FP64 (E follows the cell products' precision).
#include <algorithm>

#include "efe_device.h"

namespace {
constexpr int BK = EFE_BRICK, BX = EFE_BOX;   // edges of a brick and of a box, in nodes

// (atom, cell) -> pair
struct PairMap {
  const int32_t *box, *map;   // per atom: x0 y0 z0 nx ny nz and the place of its table
  const int64_t *off;
};

__device__ inline int pair_of(const PairMap &m, int I, int cx, int cy, int cz) {
  const int32_t *b = m.box + 6 * I;
  const int x = cx - b[0], y = cy - b[1], z = cz - b[2];
  if (x < 0 || y < 0 || z < 0 || x >= b[3] || y >= b[4] || z >= b[5]) return -1;
  return m.map[m.off[I] + x + b[3] * (y + (int64_t)b[4] * z)];
}

// What the blocks hold: E (epair: E_c per coupling pair), C (bam) or
// P^C (epair nullptr: bam is the assembled P^C, nf = 1).
struct Entries {
  NodeGrid g;
  PairMap m;
  int nf, nloc;
  const double *epair;    // [pair][local node][k]
  const double *bam;      // [support node][k]
  const int32_t *lmap;    // [pair][local node] -> support node
};

// The pairs that a box of edge e can meet, atom by atom, in LDS: nc^3 cells from
// the one before the box's first node.  Reading box, table and pair behind each
// other for every entry instead made a build of the boxes' blocks of 64 atoms take
// 1.7 ms (now 0.78).
__host__ __device__ constexpr int box_cells(int e, int p) { return (e - 1 + p - 1) / p + 2; }

__device__ __forceinline__ void box_pairs(const Entries &s, const int32_t *atom, int na,
                                          const int o[3], int nc, int32_t *tab) {
  const int n3 = nc * nc * nc;
  for (int i = threadIdx.x; i < na * n3; i += blockDim.x) {
    const int c = i % n3;
    tab[i] = pair_of(s.m, atom[i / n3], o[0] / s.g.p - 1 + c % nc, o[1] / s.g.p - 1 + c / nc % nc,
                     o[2] / s.g.p - 1 + c / (nc * nc));
  }
}

// The (up to eight) cells of a node: place in an atom's part of the table (-1:
// not a cell of the node) and the node's number there.  The cells come in the
// order of their numbers from n = 7 down.
struct NodeCells {
  int at[8], l[8];
  __device__ __forceinline__ NodeCells(const NodeGrid &g, const int o[3], const int ijk[3], int nc,
                                       bool in) {
    int cd[3], ld[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int c = ijk[d] / g.p;
      ld[d] = ijk[d] - c * g.p;
      cd[d] = c - (o[d] / g.p - 1);
    }
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int x = n & 1, y = n >> 1 & 1, z = n >> 2;
      const bool on = in && !(x && ld[0]) && !(y && ld[1]) && !(z && ld[2]);
      at[n] = on ? cd[0] - x + nc * (cd[1] - y + nc * (cd[2] - z)) : -1;
      l[n] = (x ? g.p : ld[0]) + g.P * ((y ? g.p : ld[1]) + g.P * (z ? g.p : ld[2]));
    }
  }
};

// An entry in two parts, so that several are on their way at once: request()
// the per-cell values (and the support node), then value()
struct EntryLoad {
  double e[8], b;
  int32_t sn;
  __device__ __forceinline__ void request(const Entries &s, const NodeCells &c, const int32_t *tab,
                                          int k) {
    int64_t o[8];
    int32_t q[8];
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int pr = c.at[n] >= 0 ? tab[c.at[n]] : -1;
      o[n] = pr >= 0 ? (int64_t)pr * s.nloc + c.l[n] : -1;
      e[n] = 0.0;
      q[n] = -1;
    }
    if (s.epair)
#pragma unroll
      for (int n = 0; n < 8; ++n)
        if (o[n] >= 0) e[n] = s.epair[o[n] * s.nf + k];
    sn = -1;
    if (s.bam) {
#pragma unroll
      for (int n = 0; n < 8; ++n)
        if (o[n] >= 0) q[n] = s.lmap[o[n]];
#pragma unroll
      for (int n = 0; n < 8; ++n) sn = q[n] >= 0 ? q[n] : sn;
    }
  }
  __device__ __forceinline__ void request_support(const Entries &s, int k) {
    b = sn >= 0 ? s.bam[(int64_t)sn * s.nf + k] : 0.0;
  }
  __device__ __forceinline__ double value() const {
    double v = 0.0;
#pragma unroll
    for (int n = 7; n >= 0; --n) v += e[n];
    return v + b;
  }
};

// Bricks: tile[rb][ks][lane] = entry(function 4 ks + lane/16, node 16 rb + row
// of the lane), the A operand of v_mfma_*_16x16x4.  The FP32 copy has rows
// 4 a + b and 4 b + a exchanged, so that the accumulators of both precisions
// hold the same nodes.  One wave per 16-row block.
__device__ __forceinline__ void tiles_brick(const Entries &s, int64_t b,
                                            const int32_t *__restrict__ ptr,
                                            const int32_t *__restrict__ atom,
                                            const int64_t *__restrict__ off,
                                            double *__restrict__ T64, float *__restrict__ T32,
                                            int32_t *tab /* 16 atoms */) {
  const int a0 = ptr[b], na = ptr[b + 1] - a0;
  if (na == 0) return;
  const int K = na * s.nf, KS = (K + 3) / 4;
  const int rb = threadIdx.x / 64, lane = threadIdx.x % 64, li = lane % 16, lk = lane / 16;
  const int nc = box_cells(BK, s.g.p), n3 = nc * nc * nc;
  int o[3], ijk[3];
  box_origin(s.g, BK, b, o);
  const bool in = box_node(s.g, BK, o, 16 * rb + li, ijk);
  const NodeCells cells(s.g, o, ijk, nc, in);
  const int64_t base = 256 * off[b] + (int64_t)rb * KS * 64;
  const int lp = 16 * lk + 4 * (li % 4) + li / 4;
  constexpr int U = 2;
  for (int q0 = 0; q0 < na; q0 += 16) {
    const int nq = min(16, na - q0), f0 = q0 * s.nf, ks1 = min(KS, (f0 + 16 * s.nf) / 4);
    __syncthreads();
    box_pairs(s, atom + a0 + q0, nq, o, nc, tab);
    __syncthreads();
    for (int ks = f0 / 4; ks < ks1; ks += U) {
      EntryLoad v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int f = min(4 * (ks + u) + lk, f0 + nq * s.nf - 1) - f0;
        v[u].request(s, cells, tab + f / s.nf * n3, f % s.nf);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int f = min(4 * (ks + u) + lk, f0 + nq * s.nf - 1) - f0;
        v[u].request_support(s, f % s.nf);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (ks + u >= ks1) continue;
        const double x = 4 * (ks + u) + lk < K ? v[u].value() : 0.0;
        T64[base + (int64_t)(ks + u) * 64 + lane] = x;
        if (T32) T32[base + (int64_t)(ks + u) * 64 + lp] = (float)x;
      }
    }
  }
}

// Boxes: tile[rb][ks][lane] = entry(function 16 rb + lane%16, node 4 ks +
// lane/16); live: bit c set where the nodes 16 c .. hold a non-zero entry.  One
// work-group per block and part of its nodes (1, or 4 that write a byte of live
// each), U entries of a wave in flight.
template <int U, int PARTS>
__device__ __forceinline__ void tiles_box(const Entries &s, int64_t row, int part,
                                          const int32_t *__restrict__ ptr,
                                          const int32_t *__restrict__ atom,
                                          const int32_t *__restrict__ rboff,
                                          const int32_t *__restrict__ rbbox,
                                          double *__restrict__ T64, float *__restrict__ T32,
                                          uint32_t *__restrict__ live, uint32_t &mask,
                                          int32_t *tab /* the atoms of 16 functions */) {
  const int b = rbbox[row], rb = (int)row - rboff[b];
  const int a0 = ptr[b], na = ptr[b + 1] - a0, K = na * s.nf;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, li = lane % 16, lk = lane / 16;
  const int f = 16 * rb + li, q0 = 16 * rb / s.nf, k = f % s.nf;
  const int nc = box_cells(BX, s.g.p), n3 = nc * nc * nc;
  int o[3], ijk[3];
  box_origin(s.g, BX, b, o);
  if (threadIdx.x == 0) mask = 0;
  box_pairs(s, atom + a0 + q0, min((16 * rb + 15) / s.nf + 1, na) - q0, o, nc, tab);
  __syncthreads();
  const int32_t *const ft = tab + (f / s.nf - q0) * n3;
  constexpr int KS = BX * BX * BX / 4, KP = KS / PARTS;
  static_assert(KS / 4 == 32 && (PARTS == 1 || PARTS == 4) && KP % (4 * U) == 0, "a byte a part");
  for (int ks = part * KP + wave; ks < (part + 1) * KP; ks += 4 * U) {
    EntryLoad v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = box_node(s.g, BX, o, 4 * (ks + 4 * u) + lk, ijk);
      v[u].request(s, NodeCells(s.g, o, ijk, nc, in && f < K), ft, k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) v[u].request_support(s, k);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double x = v[u].value();
      const int64_t at = (row * KS + ks + 4 * u) * 64 + lane;
      T64[at] = x;
      if (T32) T32[at] = (float)x;
      if (__ballot(x != 0.0) && lane == 0) atomicOr(&mask, 1u << ((ks + 4 * u) / 4 - KP / 4 * part));
    }
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (PARTS == 1) live[row] = mask;
  else ((uint8_t *)live)[PARTS * row + part] = (uint8_t)mask;
}

// Both sets of one family of functions.  Few blocks (TILES_FEW): four work-groups a
// block of a box, four entries in flight, and the bricks in the same launch, which
// shortens the chain of loads (27 boxes: 15.6 us, 57 as below); many: two launches,
// one work-group a block, two entries in flight, whose registers leave more waves
// to cover the loads (64 atoms: 1.05 ms, 1.23 as above).
constexpr int64_t TILES_FEW = 512;
struct TileArgs {
  Entries s;
  const int32_t *bx_ptr, *bx_atom, *rboff, *rbbox, *bk_ptr, *bk_atom;
  const int64_t *bk_off;
  double *T1, *T2;
  float *T1f, *T2f;
  uint32_t *live;
  int64_t n_rb;
};
template <int U, int PARTS, bool BRICKS>
__global__ __launch_bounds__(256) void k_tiles(TileArgs a) {
  __shared__ uint32_t mask;
  extern __shared__ int32_t tab[];
  const int64_t b = blockIdx.x, nb = PARTS * a.n_rb;
  if constexpr (PARTS > 0)
    if (b < nb) {
      tiles_box<U, PARTS>(a.s, b / PARTS, (int)(b % PARTS), a.bx_ptr, a.bx_atom, a.rboff, a.rbbox,
                          a.T2, a.T2f, a.live, mask, tab);
      return;
    }
  if constexpr (BRICKS)
    tiles_brick(a.s, b - nb, a.bk_ptr, a.bk_atom, a.bk_off, a.T1, a.T1f, tab);
}

// Second part of H^E_ee = H^phiphi - C B^T - E C^T (the first: k_hee_rows,
// setup.hip): -E C^T as products of the box blocks of E with C.  One work-group
// takes a box and 16 functions of C (its nodes x 16 in LDS as the B operand), each
// wave every fourth row block, and only the chunks of 16 nodes in which both have
// entries; the 16 x 16 results are added into Hee atomically (64 atoms: 2.6 ms;
// 4.2 with all chunks; 32 functions a work-group read E half as often but leave
// one work-group a CU, whose fill of C nothing covers, 3.1).  gridDim.y parts of
// the nodes: with few blocks (HEE_FEW) eight, whose loads behind each other are an
// eighth (27 boxes: 56 us in one part); with many one, as every part adds its own
// products atomically.
constexpr int64_t HEE_FEW = 512;
typedef double v4d_c __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void k_hee_box(Entries s, const int32_t *__restrict__ ptr,
                                                 const int32_t *__restrict__ atom,
                                                 const int32_t *__restrict__ rboff,
                                                 const int32_t *__restrict__ rbbox,
                                                 const double *__restrict__ T,
                                                 const uint32_t *__restrict__ live,
                                                 const double *__restrict__ C_am, int64_t n_enr,
                                                 double *__restrict__ Hee) {
  constexpr int NB = BX * BX * BX, KS = NB / 4, U = 2;
  __shared__ double Cs[NB][16];
  __shared__ uint32_t cmask;
  extern __shared__ int32_t tab[];
  const int64_t row = blockIdx.x;
  const int b = rbbox[row], cb = (int)row - rboff[b], nrb = rboff[b + 1] - rboff[b];
  const int a0 = ptr[b], na = ptr[b + 1] - a0, K = na * s.nf, q0 = 16 * cb / s.nf;
  const int nc = box_cells(BX, s.g.p), n3 = nc * nc * nc;
  int o[3];
  box_origin(s.g, BX, b, o);
  Entries c = s;
  c.epair = nullptr;
  c.bam = C_am;
  if (threadIdx.x == 0) cmask = 0;
  box_pairs(s, atom + a0 + q0, min((16 * cb + 15) / s.nf + 1, na) - q0, o, nc, tab);
  __syncthreads();
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, li = lane % 16, lk = lane / 16;
  const int f2 = 16 * cb + li;
  const int32_t *const ft = tab + (f2 / s.nf - q0) * n3;
  const int ksp = KS / (int)gridDim.y, ks0 = (int)blockIdx.y * ksp;
  for (int ks = ks0 + wave; ks < ks0 + ksp; ks += 4 * U) {
    EntryLoad v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int ijk[3];
      const bool in = box_node(s.g, BX, o, 4 * (ks + 4 * u) + lk, ijk);
      v[u].request(c, NodeCells(s.g, o, ijk, nc, in && f2 < K), ft, f2 % s.nf);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) v[u].request_support(c, f2 % s.nf);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double x = v[u].value();
      Cs[4 * (ks + 4 * u) + lk][li] = x;
      if (__ballot(x != 0.0) && lane == 0) atomicOr(&cmask, 1u << ((ks + 4 * u) / 4));
    }
  }
  __syncthreads();
  const uint32_t cm = __builtin_amdgcn_readfirstlane(cmask);
  const int64_t g2 = f2 < K ? (int64_t)atom[a0 + f2 / s.nf] * s.nf + f2 % s.nf : 0;
  for (int rb = __builtin_amdgcn_readfirstlane(wave); rb < nrb; rb += 4) {
    uint32_t left = live[rboff[b] + rb] & cm;
    if (left == 0) continue;
    const double *tp = T + ((int64_t)(rboff[b] + rb) * KS) * 64 + lane;
    v4d_c acc = {0.0, 0.0, 0.0, 0.0};
    double a[4], nx[4];
    int ch = __builtin_ctz(left);
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = tp[(4 * ch + i) * 64];
    while (true) {
      left &= left - 1;
      const int n = left ? __builtin_ctz(left) : ch;   // the last one requests itself again
#pragma unroll
      for (int i = 0; i < 4; ++i) nx[i] = tp[(4 * n + i) * 64];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], Cs[4 * (4 * ch + i) + lk][li], acc, 0, 0, 0);
      if (!left) break;
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = nx[i];
      ch = n;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int f1 = 16 * rb + 4 * v + lk;
      if (f1 < K && f2 < K)
        atomicAdd(&Hee[((int64_t)atom[a0 + f1 / s.nf] * s.nf + f1 % s.nf) * n_enr + g2], -acc[v]);
    }
  }
}

// Matrix of the dense part of an apply (apply.hip) over the coefficients
// (I, k), k < nf the enrichment functions and (with projectors) k = nf the
// projector of atom I: [[H^E_ee + P~^T D P~, P~^T D], [D P~, D]]; Hee holds the
// projector term already, and is symmetrized here.
__global__ void k_coef_matrix(int natoms, int nf, int nx, const double *__restrict__ Hee,
                              const double *__restrict__ Pt, const double *__restrict__ D,
                              double *__restrict__ S) {
  const int64_t n = (int64_t)natoms * nx, ne = (int64_t)natoms * nf;
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n * n) return;
  const int64_t r = i / n, c = i % n;
  const int64_t I = r / nx, J = c / nx;
  const int k = (int)(r % nx), l = (int)(c % nx);
  double v;
  if (k < nf && l < nf) {
    const int64_t f = I * nf + k, h = J * nf + l;
    v = 0.5 * (Hee[f * ne + h] + Hee[h * ne + f]);
  }
  else if (k < nf) v = Pt[J * ne + I * nf + k] * D[J];
  else if (l < nf) v = Pt[I * ne + J * nf + l] * D[I];
  else v = I == J ? D[I] : 0.0;
  S[i] = v;
}

// ------------------------------------------------------------------ host
// Tables of the coupling, copied to the device in one piece (two atoms on 6^3 to 8^3
// cells: setup 1.3 to 1.4 ms; with about thirty copies and waits of their own 1.5 to 1.8)
struct Pack {
  std::vector<char> host;
  std::vector<std::pair<void **, size_t>> at;
  template <class T>
  void add(T **dst, const std::vector<T> &v) {
    const size_t o = (host.size() + 255) & ~(size_t)255;
    host.resize(o + std::max<size_t>(v.size(), 1) * sizeof(T));
    std::copy((const char *)v.data(), (const char *)(v.data() + v.size()), host.data() + o);
    at.push_back({(void **)dst, o});
  }
  efe_status upload(efe_ctx *c, char **base) {
    efe_status s = efe_alloc(c, (void **)base, host.size());
    if (s) return s;
    HIPCHK(c, hipMemcpyAsync(*base, host.data(), host.size(), hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    for (auto &a : at) *a.first = *base + a.second;
    return EFE_OK;
  }
};

// atoms touching every box of edge e (ascending), from each atom's cells
void box_atoms(const efe_ctx *c, const std::vector<int32_t> &ptr, const std::vector<int32_t> &cells,
               int e, std::vector<int32_t> &bptr, std::vector<int32_t> &batom) {
  const NodeGrid g = node_grid(c);
  const int nb[3] = {(g.n1[0] + e - 1) / e, (g.n1[1] + e - 1) / e, (g.n1[2] + e - 1) / e};
  const int64_t n = (int64_t)nb[0] * nb[1] * nb[2];
  std::vector<int32_t> mark(n, -1), list, lptr(c->natoms + 1, 0);
  bptr.assign(n + 1, 0);
  for (int I = 0; I < c->natoms; ++I) {
    for (int32_t q = ptr[I]; q < ptr[I + 1]; ++q) {
      const int32_t cl = cells[q];
      const int cc[3] = {cl % g.nc[0], (cl / g.nc[0]) % g.nc[1], cl / (g.nc[0] * g.nc[1])};
      int lo[3], hi[3];   // boxes of the cell's interior nodes
      for (int d = 0; d < 3; ++d) {
        lo[d] = std::max(cc[d] * g.p, 1) / e;
        hi[d] = std::min(cc[d] * g.p + g.p, g.n1[d] - 2) / e;
      }
      for (int z = lo[2]; z <= hi[2]; ++z)
        for (int y = lo[1]; y <= hi[1]; ++y)
          for (int x = lo[0]; x <= hi[0]; ++x) {
            const int64_t b = x + nb[0] * (y + (int64_t)nb[1] * z);
            if (mark[b] == I) continue;
            mark[b] = I;
            list.push_back((int32_t)b);
            bptr[b + 1]++;
          }
    }
    lptr[I + 1] = (int32_t)list.size();
  }
  for (int64_t b = 0; b < n; ++b) bptr[b + 1] += bptr[b];
  batom.resize(list.size());
  std::vector<int32_t> fill(bptr.begin(), bptr.end() - 1);
  for (int I = 0; I < c->natoms; ++I)
    for (int32_t q = lptr[I]; q < lptr[I + 1]; ++q) batom[fill[list[q]]++] = I;
}

void build_set(const efe_ctx *c, const std::vector<int32_t> &ptr, const std::vector<int32_t> &cells,
               int nf, CoupleSet &S, Pack &pk) {
  S.nf = nf;
  // (atom, cell) -> pair over the bounding box of the atom's cells
  std::vector<int32_t> box(6 * (size_t)c->natoms, 0), map;
  std::vector<int64_t> off(c->natoms + 1, 0);
  for (int I = 0; I < c->natoms; ++I) {
    int lo[3] = {1 << 30, 1 << 30, 1 << 30}, hi[3] = {-1, -1, -1};
    auto ijk = [&](int32_t cl, int d) {
      return d == 0 ? cl % c->ncell[0]
                    : d == 1 ? (cl / c->ncell[0]) % c->ncell[1] : cl / (c->ncell[0] * c->ncell[1]);
    };
    for (int32_t q = ptr[I]; q < ptr[I + 1]; ++q)
      for (int d = 0; d < 3; ++d) {
        lo[d] = std::min(lo[d], ijk(cells[q], d));
        hi[d] = std::max(hi[d], ijk(cells[q], d));
      }
    int64_t n = ptr[I + 1] > ptr[I] ? 1 : 0;
    for (int d = 0; d < 3 && n; ++d) {
      box[6 * I + d] = lo[d];
      box[6 * I + 3 + d] = hi[d] - lo[d] + 1;
      n *= hi[d] - lo[d] + 1;
    }
    off[I + 1] = off[I] + n;
    map.resize(off[I + 1], -1);
    for (int32_t q = ptr[I]; q < ptr[I + 1]; ++q)
      map[off[I] + (ijk(cells[q], 0) - lo[0]) +
          (int64_t)box[6 * I + 3] * ((ijk(cells[q], 1) - lo[1]) +
                                     (int64_t)box[6 * I + 4] * (ijk(cells[q], 2) - lo[2]))] = q;
  }
  pk.add(&S.d_box, box);
  pk.add(&S.d_map, map);
  pk.add(&S.d_off, off);
  // bricks
  std::vector<int32_t> bptr, batom;
  box_atoms(c, ptr, cells, BK, bptr, batom);
  std::vector<int64_t> ksoff(bptr.size(), 0);
  for (size_t b = 0; b + 1 < bptr.size(); ++b)
    ksoff[b + 1] = ksoff[b] + cdiv((int64_t)(bptr[b + 1] - bptr[b]) * nf, 4);
  S.n_brick = (int64_t)bptr.size() - 1;
  S.brick_tile = 256 * ksoff.back();
  pk.add(&S.d_bk_ptr, bptr);
  pk.add(&S.d_bk_atom, batom);
  pk.add(&S.d_bk_off, ksoff);
  // boxes
  box_atoms(c, ptr, cells, BX, bptr, batom);
  std::vector<int32_t> rboff(bptr.size(), 0), rbbox;
  for (size_t b = 0; b + 1 < bptr.size(); ++b) {
    const int n = (int)cdiv((int64_t)(bptr[b + 1] - bptr[b]) * nf, 16);
    rboff[b + 1] = rboff[b] + n;
    rbbox.insert(rbbox.end(), n, (int32_t)b);
  }
  S.n_box = (int64_t)bptr.size() - 1;
  S.n_boxpairs = (int64_t)batom.size();
  S.n_rb = rboff.back();
  S.h_rboff = rboff;
  pk.add(&S.d_live, std::vector<uint32_t>(S.n_rb, 0));
  S.box_tile = S.n_rb * (BX * BX * BX / 4) * 64;
  std::vector<int32_t> aptr(c->natoms + 1, 0), apos(batom.size());
  for (int32_t a : batom) aptr[a + 1]++;
  for (int I = 0; I < c->natoms; ++I) aptr[I + 1] += aptr[I];
  std::vector<int32_t> fill(aptr.begin(), aptr.end() - 1);
  for (size_t q = 0; q < batom.size(); ++q) apos[fill[batom[q]]++] = (int32_t)q;
  pk.add(&S.d_bx_ptr, bptr);
  pk.add(&S.d_bx_atom, batom);
  pk.add(&S.d_rboff, rboff);
  pk.add(&S.d_rbbox, rbbox);
  pk.add(&S.d_at_ptr, aptr);
  pk.add(&S.d_at_pos, apos);
}

Entries entries(const efe_ctx *c, const CoupleSet &S, const double *epair, const double *bam,
                const int32_t *lmap) {
  return {node_grid(c), {S.d_box, S.d_map, S.d_off}, S.nf, c->nloc, epair, bam, lmap};
}
// LDS of the pair tables: 16 atoms of a brick, the atoms of 16 functions of a box
size_t brick_lds(const efe_ctx *c) {
  const int n = box_cells(BK, c->p);
  return 16 * (size_t)(n * n * n) * 4;
}
size_t box_lds(int p, int nf) {
  const int n = box_cells(BX, p);
  return std::min(16, 14 / nf + 2) * (size_t)(n * n * n) * 4;
}
void launch_tiles(efe_ctx *c, const CoupleSet &S, const Entries &e, bool f32) {
  const TileArgs a{e,         S.d_bx_ptr, S.d_bx_atom, S.d_rboff, S.d_rbbox, S.d_bk_ptr,
                   S.d_bk_atom, S.d_bk_off, S.d_T1,      S.d_T2,    f32 ? S.d_T1f : nullptr,
                   f32 ? S.d_T2f : nullptr, S.d_live, S.n_rb};
  const size_t l1 = brick_lds(c), l2 = box_lds(c->p, S.nf);
  if (S.n_rb < TILES_FEW) {
    k_tiles<4, 4, true><<<4 * S.n_rb + S.n_brick, 256, std::max(l1, l2), c->stream>>>(a);
    return;
  }
  k_tiles<2, 1, false><<<S.n_rb, 256, l2, c->stream>>>(a);
  k_tiles<2, 0, true><<<S.n_brick, 256, l1, c->stream>>>(a);
}
}  // namespace

// Work items of the box products: four consecutive 16-row blocks of a box, E
// blocks first, then P^C blocks, as (box, first block); the last three lists
// are E only, P^C only and both.
efe_status efe_couple_setup(efe_ctx *c, const std::vector<int32_t> &eptr,
                            const std::vector<int32_t> &ecells) {
  efe_status s;
  CoupleSet &E = c->cpl_e, &K = c->cpl_k;
  // the same bound for every context: what the lowest order and one function an
  // atom need
  HIPCHK(c, hipFuncSetAttribute((const void *)k_hee_box, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)box_lds(1, 1)));
  const std::vector<int32_t> none(c->natoms + 1, 0);
  Pack pk;
  build_set(c, c->nf > 0 ? eptr : none, ecells, std::max(c->nf, 1), E, pk);
  build_set(c, c->nproj ? c->kb_ptr : none, c->kb_cells, 1, K, pk);
  std::vector<int32_t> items[3];
  for (int64_t b = 0; b < E.n_box; ++b) {
    const int ne = E.h_rboff[b + 1] - E.h_rboff[b], nk = K.h_rboff[b + 1] - K.h_rboff[b];
    for (int which = 0; which < 3; ++which) {
      const int r0 = which == 1 ? ne : 0, r1 = which == 0 ? ne : ne + nk;
      for (int r = r0; r < r1; r += 4) {
        items[which].push_back((int32_t)b);
        items[which].push_back(r);
      }
    }
  }
  for (int which = 0; which < 3; ++which) {
    c->n_items[which] = (int64_t)items[which].size() / 2;
    pk.add(&c->d_items[which], items[which]);
  }
  if ((s = pk.upload(c, &c->d_cpl))) return s;
  if (c->nproj) {
    if ((s = efe_alloc(c, (void **)&K.d_T1, std::max<int64_t>(K.brick_tile, 1) * 8))) return s;
    if ((s = efe_alloc(c, (void **)&K.d_T2, std::max<int64_t>(K.box_tile, 1) * 8))) return s;
  }
  return EFE_OK;
}

// blocks of P^C (once, when the projectors are known)
efe_status efe_couple_projectors(efe_ctx *c) {
  CoupleSet &K = c->cpl_k;
  if (!c->nproj || K.n_boxpairs == 0) return EFE_OK;
  const Entries e = entries(c, K, nullptr, c->d_Pc_am, c->d_kbpair_lmap);
  launch_tiles(c, K, e, false);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}

// memory of efe_couple_build
efe_status efe_couple_alloc(efe_ctx *c, bool want32) {
  efe_status s;
  CoupleSet &E = c->cpl_e;
  const int64_t n = (int64_t)c->natoms * (c->nf + (c->nproj ? 1 : 0));
  if (n == 0) return EFE_OK;
  if (!c->d_S && (s = efe_alloc(c, (void **)&c->d_S, n * n * 8))) return s;
  if (c->nf == 0 || E.n_boxpairs == 0) return EFE_OK;
  if (!E.d_T1 && (s = efe_alloc(c, (void **)&E.d_T1, E.brick_tile * 8))) return s;
  if (!E.d_T2 && (s = efe_alloc(c, (void **)&E.d_T2, E.box_tile * 8))) return s;
  if (want32 && !E.d_T1f && (s = efe_alloc(c, (void **)&E.d_T1f, E.brick_tile * 4))) return s;
  if (want32 && !E.d_T2f && (s = efe_alloc(c, (void **)&E.d_T2f, E.box_tile * 4))) return s;
  return EFE_OK;
}

// blocks of E from the per-cell E_c (d_Epair), H^E_ee and the matrix of the
// coefficients, for a new potential
efe_status efe_couple_build(efe_ctx *c, bool want32) {
  CoupleSet &E = c->cpl_e;
  const int64_t ne = c->n_enr;
  const int nx = c->nf + (c->nproj ? 1 : 0);
  const int64_t n = (int64_t)c->natoms * nx;
  if (n == 0) return EFE_OK;
  if (c->nf > 0 && E.n_boxpairs > 0) {
    const Entries e = entries(c, E, c->d_Epair, nullptr, c->d_cpair_lmap);
    launch_tiles(c, E, e, want32);
    if (c->max_rbe > 2)   // else k_build_E forms E C^T
      k_hee_box<<<dim3(E.n_rb, E.n_rb < HEE_FEW ? 8 : 1), 256, box_lds(c->p, c->nf), c->stream>>>(
        e, E.d_bx_ptr, E.d_bx_atom, E.d_rboff, E.d_rbbox, E.d_T2, E.d_live, c->d_C_am, ne, c->d_Hee);
  }
  k_coef_matrix<<<cdiv(n * n, 256), 256, 0, c->stream>>>(c->natoms, c->nf, nx, c->d_Hee, c->d_Ptil,
                                                        c->d_D, c->d_S);
  HIPCHK(c, hipGetLastError());
  return EFE_OK;
}

void efe_couple_free(efe_ctx *c) {
  for (CoupleSet *S : {&c->cpl_e, &c->cpl_k}) {
    void *ptrs[] = {S->d_T1, S->d_T2, S->d_T1f, S->d_T2f};
    for (void *p : ptrs) efe_free(c, p);
  }
  efe_free(c, c->d_cpl);   // every table
}
