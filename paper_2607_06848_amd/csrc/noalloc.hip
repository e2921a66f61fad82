// Chebyshev filter that allocates nothing, for callers that cannot call the
// device allocator (code under stream capture, tight serving loops).  Its
// workspaces come from `scratch`, a fixed region of device memory that every
// GPU the library runs on holds until the process ends; its address on each
// device is taken once, when the first context on that device is set up.
#include <mutex>

#include "efe_internal.h"

static __device__ __align__(256) unsigned char scratch[EFE_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {nullptr};
}  // namespace

efe_status efe_scratch_attach(efe_ctx *c) {
  if (c->device < 0 || c->device >= kMaxDevices) EFE_FAIL(c, EFE_EINVAL, "device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[c->device]) return EFE_OK;
  // the context's device is the current one here (efe_setup_mesh)
  void *p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p) {
    c->err = std::string("hipGetSymbolAddress of the scratch region failed: ") + hipGetErrorString(e);
    return EFE_EHIP;
  }
  g_scratch_ptr[c->device] = p;
  return EFE_OK;
}

// Workspace bytes that a filter call is accepted by: G, Z_{k-1}, Z_{k-2}, H V,
// the enrichment rows of M~^-1 Z, the C_k(lambda) and sigma tables; per apply
// copies of the CFE and enrichment rows, projector coefficients, one partial
// row per (cell, enrichment function) and dense-block products; 256-byte
// alignment of every slot.
static size_t filter_accept_bytes(const efe_ctx *c, int32_t ncols, int m) {
  const size_t nc = (size_t)std::min<int32_t>(ncols, EFE_COL_CHUNK);
  const size_t ldc = (nc + 1) & ~(size_t)1;
  const size_t rows = (size_t)c->rows, nn = (size_t)c->n_nodes;
  const size_t ne = (size_t)c->n_enr, ne1 = std::max<size_t>(ne, 1);
  size_t b = 4 * rows * nc * 8 + ne1 * nc * 8 + (size_t)(m + 1) * nc * 8 + (size_t)(m + 1) * 8;
  b += nn * ldc * 8 + ne * ldc * 8 + (size_t)c->nproj * nc * 8 +
       (size_t)c->nf * (size_t)std::max<int64_t>(c->ncpairs, 1) * nc * 8 + ne * nc * 8;
  return b + 16 * 256;
}

// Workspace bytes that the slots of a chunk of nc columns take (the first
// chunk is the widest), without the cells' products, which may be missing
static size_t filter_chunk_bytes(const efe_ctx *c, size_t nc, int m) {
  const size_t ldc = (nc + 1) & ~(size_t)1;
  const size_t rows = (size_t)c->rows, ne1 = std::max<size_t>((size_t)c->n_enr, 1);
  const size_t nq = (size_t)c->natoms * (c->nf + (c->nproj ? 1 : 0)) + c->nproj;
  const size_t np = (size_t)std::max<int64_t>(
      (c->nf > 0 ? c->nf * c->cpl_e.n_boxpairs : 0) + c->cpl_k.n_boxpairs, 1);
  size_t b = 4 * rows * nc * 8 + ne1 * nc * 8 + (size_t)(m + 1) * nc * 8 + (size_t)(m + 1) * 8;
  b += (nq + ne1) * ldc * 8 + np * nc * 8;
  if (!c->tp || c->have16) b += (size_t)c->n_nodes * ldc * 8;
  return b + 16 * 256;
}

extern "C" efe_status efe_cheb_filter_noalloc(efe_ctx *c, double *V, const double *lambda,
                                              int32_t ncols, int64_t ld,
                                              const efe_cheb_params *prm) {
  efe_status s = efe_filter_check(c, V, lambda, ncols, ld, prm);
  if (s) return s;
  void *base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (c->device >= 0 && c->device < kMaxDevices) base = g_scratch_ptr[c->device];
  }
  if (!base) EFE_FAIL(c, EFE_ESTATE, "no scratch region on this device");
  const size_t need = filter_accept_bytes(c, ncols, prm->degree);
  if (need > (size_t)EFE_NOALLOC_SCRATCH_BYTES)
    EFE_FAIL(c, EFE_EINVAL,
             "filter needs " + std::to_string(need) + " bytes of scratch, more than the " +
                 std::to_string((size_t)EFE_NOALLOC_SCRATCH_BYTES) + " the region holds");
  // every workspace slot from the region; timing would create events, so it
  // is off for the call
  const bool timing = c->timing;
  c->timing = false;
  c->arena = (char *)base;
  c->arena_cap = EFE_NOALLOC_SCRATCH_BYTES;
  c->arena_used = 0;
  // the slots differ from what a call is accepted by: where they are larger (atoms
  // on a handful of nodes), the columns go through in narrower chunks
  c->col_chunk = std::min<int32_t>(std::max<int32_t>(ncols, 1), EFE_COL_CHUNK);
  while (c->col_chunk > 1 && filter_chunk_bytes(c, c->col_chunk, prm->degree) > c->arena_cap)
    c->col_chunk = (c->col_chunk + 1) / 2;
  c->arena_spare =
      c->arena_cap - std::min(c->arena_cap, filter_chunk_bytes(c, c->col_chunk, prm->degree));
  for (int i = 0; i < efe_ctx::kArenaSlots; ++i) c->arena_len[i] = 0;
  s = efe_filter_run(c, V, lambda, ncols, ld, prm);
  c->arena = nullptr;
  c->arena_cap = 0;
  c->col_chunk = EFE_COL_CHUNK;
  c->timing = timing;
  return s;
}
