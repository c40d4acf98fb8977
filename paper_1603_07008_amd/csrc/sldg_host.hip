// Host side of libsldg: the C ABI declared in include/sldg.h -- plans,
// argument validation, per-line tables and kernel launches for the sLdG
// projection sweep (L. Einkemmer, arXiv 1603.07008, section II-A).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

#include "sldg.h"
#include "sldg_internal.h"
#include "sldg_ref.h"
#include "sldg_field.h"
#include "sldg_colloc.h"
#include "sldg_fused.h"
#include "sldg_strang.h"
#include "sldg_colpair.h"
#include "sldg_colsweep.h"
#include "sldg_line.h"

using namespace sldg;

struct sldg_plan_s {
  int ndim;
  int64_t n[kMaxDim];
  int k, o;
  sldg_tier tier;
  hipStream_t stream;
  int device;
  int64_t cells;
  int64_t modes;          // o^ndim
  int ndouble;            // modes of total degree < ndouble are stored in FP64
  int64_t n_lo, n_hi;     // planes in the FP64 array and in the storage-type array
  int64_t lo_bytes;
  int64_t hi_bytes;
  int32_t* d_pmap;        // per mode: >= 0 hi plane, < 0 lo plane -1-v
  std::vector<int32_t> h_pmap;
  int64_t table_cap;      // entries of the per-line table
  int32_t* d_s;
  double* d_ab;
  int mass_nblocks;
  double* d_mass_part;    // [2 * mass_nblocks]
  double* d_mass_out;     // [2]
  double* h_mass_out;     // pinned [2]
  // launch shape of the sweeps along each dimension
  int rows_d[kMaxDim];    // strided sweep: rows per thread (1, 2, 4 or 8)
  int tuples_d[kMaxDim];  // spectator tuples per thread (0: all)
  int colwaves_d[kMaxDim];// strided sweep: waves of a workgroup along the columns (1, 2, 4)
  int xcd_contig;         // XCD-aware tile order (run length) of the dimension-0 sweep
  int xcd_strided;        // ... and of the strided sweeps
  // fused pair of sweeps along dimensions 0 and 1 (sldg_advect_dims01)
  int fuse;               // split steps fuse eligible (0, 1) pairs
  int xy_rows;            // tile rows of dimension 1 (0: the most that fit)
  int xcd_xy;             // XCD-aware tile order of the fused pass
  int xcd_strang;         // ... and of the X V X pass
  // scaled FP16 storage
  int scale_headroom;     // binades between a plane's absmax and 2^15
  int32_t* d_hmode;       // [n_hi] mode id of every hi plane
  int32_t* d_redo;        // [n_hi] planes to recompute after a scaled sweep, then their count
  float* d_part;          // absmax partials, grown on demand
  int64_t part_cap;       // floats in d_part
  double* d_field;        // scratch of the field solve, grown on demand
  int64_t field_cap;      // doubles in d_field
  // kernel timing (sldg_timing_*)
  bool timing;
  int ntimed;
  hipEvent_t ev[2 * 4096];
  int ev_dim[4096];
  int nev_created;
};

// Device memory of the allocation-free field solve (sldg_poisson_shift_noalloc):
// a fixed array in the library's code object, one copy per device, held until
// the process ends.  Host code never passes `scratch` itself to a kernel (on
// the host it is only a stand-in for the symbol): it looks up each device's
// address once, with hipGetSymbolAddress, and uses that.
constexpr int64_t kStaticFieldDoubles = int64_t(1) << 19;    // 4 MiB
static __device__ __align__(256) double scratch[kStaticFieldDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

namespace sldg {

static thread_local char g_err[512] = "";

sldg_status fail(sldg_status st, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
  return st;
}

sldg_status ok() {
  g_err[0] = '\0';
  return SLDG_OK;
}

const char* last_error_text() { return g_err; }

int64_t elem_size(sldg_tier t) {
  switch (t) {
    case SLDG_TIER_FP64: return 8;
    case SLDG_TIER_FP32: return 4;
    case SLDG_TIER_BF16: return 2;
    case SLDG_TIER_FP16: return 2;
  }
  return 0;
}

bool overlap(const void* a, int64_t na, const void* b, int64_t nb) {
  const char* pa = static_cast<const char*>(a);
  const char* pb = static_cast<const char*>(b);
  return pa < pb + nb && pb < pa + na;
}

sldg_status device_error(hipError_t e, const char* what) {
  return fail(SLDG_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

namespace {
std::mutex g_alloc_mu;
int64_t g_alloc_limit = -1;                    // bytes; -1: no limit
int64_t g_alloc_live = 0;                      // bytes held by live allocations
std::unordered_map<void*, size_t> g_alloc_size;
}  // namespace

hipError_t dev_malloc_raw(void** p, size_t bytes) {
  std::lock_guard<std::mutex> lock(g_alloc_mu);
  *p = nullptr;
  if (g_alloc_limit >= 0 && g_alloc_live + (int64_t)bytes > g_alloc_limit)
    return hipErrorOutOfMemory;
  const hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    return e;
  }
  g_alloc_size[*p] = bytes;
  g_alloc_live += (int64_t)bytes;
  return hipSuccess;
}

void dev_free(void* p) {
  if (!p) return;
  {
    std::lock_guard<std::mutex> lock(g_alloc_mu);
    auto it = g_alloc_size.find(p);
    if (it != g_alloc_size.end()) {
      g_alloc_live -= (int64_t)it->second;
      g_alloc_size.erase(it);
    }
  }
  (void)hipFree(p);
}

bool dev_alloc_fits(int64_t bytes) {
  std::lock_guard<std::mutex> lock(g_alloc_mu);
  return g_alloc_limit < 0 || g_alloc_live + bytes <= g_alloc_limit;
}

bool dev_alloc_limited() {
  std::lock_guard<std::mutex> lock(g_alloc_mu);
  return g_alloc_limit >= 0;
}

void describe_grid(int ndim, const int64_t* n, int o, int64_t modes, int dim, uint32_t dep_mask,
                   int rows_per_thread, int tuples_per_thread, SweepArgs& a, int64_t& ntab) {
  int64_t P = 1, Q = 1, cells = 1;
  for (int e = 0; e < ndim; ++e) cells *= n[e];
  for (int e = 0; e < dim; ++e) P *= n[e];
  for (int e = dim + 1; e < ndim; ++e) Q *= n[e];
  a.cells = cells;
  a.P = (int32_t)P;
  a.N = (int32_t)n[dim];
  a.Q = (int32_t)Q;
  int64_t ms = 1;
  for (int e = 0; e < dim; ++e) ms *= o;
  a.mstride = (int32_t)ms;
  a.nspec = (int32_t)(modes / o);
  // table over the dependent dims, lowest fastest
  LineMap m{};
  int64_t str = 1, div_lo = 1, div_hi = 1;
  for (int e = 0; e < ndim; ++e) {
    if (e == dim) continue;
    const bool below = e < dim;
    if (dep_mask & (1u << e)) {
      if (below) {
        m.lo_div[m.nlo] = FastDiv::make((uint32_t)div_lo);
        m.lo_mod[m.nlo] = FastDiv::make((uint32_t)n[e]);
        m.lo_str[m.nlo] = (int32_t)str;
        ++m.nlo;
      } else {
        m.hi_div[m.nhi] = FastDiv::make((uint32_t)div_hi);
        m.hi_mod[m.nhi] = FastDiv::make((uint32_t)n[e]);
        m.hi_str[m.nhi] = (int32_t)str;
        ++m.nhi;
      }
      str *= n[e];
    }
    if (below) div_lo *= n[e];
    else div_hi *= n[e];
  }
  a.map = m;
  ntab = str;
  a.tuples = (tuples_per_thread > 0 && tuples_per_thread < a.nspec) ? tuples_per_thread : a.nspec;
  a.colwaves = 1;
  // dimension 0 without the window form: rows 1 asks for the lane form, 0
  // for the automatic choice, anything else for the group form.  The
  // automatic choice runs every tuple in one run (a thread's share of a
  // tuple is small, the run amortises the line's table), in the group form
  // when the displacement depends on dimension 1 (every line its own table,
  // shared by a group's 4 cells), else in the lane form
  a.lane = 0;
  if (dim == 0) {
    if (rows_per_thread == 1) {
      a.lane = 1;
    } else if (rows_per_thread == 0) {
      a.lane = (dep_mask & 2u) ? 0 : 1;
      a.tuples = a.nspec;
    }
  } else if (rows_per_thread == 0) {
    a.lane = 1;               // strided sweep in the lane form (one cell per lane)
  }
  // strided sweep: rows per thread (one-shot chunks along the swept dim)
  if (dim > 0) {
    int rows = a.lane ? 1 : rows_per_thread;
    while (rows > 1 && rows > a.N) rows >>= 1;
    a.chunk = rows;
    a.nchunk = (int32_t)((a.N + rows - 1) / rows);
  } else {
    a.chunk = a.N;
    a.nchunk = 1;
  }
  // non-temporal stores where every store of a wave writes whole 128-byte
  // lines: dimension 0 (consecutive lanes on consecutive cells; the group
  // form stores without the hint), and strided sweeps whose 64 columns of a
  // wave are one run (P % 64 == 0) or runs of whole lines (P * size % 128 == 0)
  a.ntmask = 0;
  for (int b = 0; b < 3; ++b) {
    const int64_t size = 2LL << b;           // 2, 4, 8 bytes
    if (dim == 0 || a.lane || P % 64 == 0 || (P * size) % 128 == 0) a.ntmask |= 1 << b;
  }
  a.fP = FastDiv::make((uint32_t)a.P);
  a.fN = FastDiv::make((uint32_t)a.N);
  a.fchunk = FastDiv::make((uint32_t)a.nchunk);
  a.fG = FastDiv::make((uint32_t)((a.N + 3) / 4));
}

}  // namespace sldg

namespace {

constexpr int kMaxTimed = 4096;
constexpr int kXYTimingDim = -3;   // timing code of the fused (0, 1) pair
constexpr int kPairTimingDim = 1 << 16;   // ... of the fused pairs along higher ones: of no single one

sldg_status check_sweep(const sldg_plan_s* p, int dim, const double* shift, uint32_t dep_mask,
                        const double* in_lo, const void* in_hi, const double* out_lo,
                        const void* out_hi) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (dim < 0 || dim >= p->ndim)
    return fail(SLDG_ERR_ARG, "dim %d out of range [0, %d)", dim, p->ndim);
  if (dep_mask >> p->ndim)
    return fail(SLDG_ERR_ARG, "dep_mask 0x%x names dimensions beyond ndim=%d", dep_mask, p->ndim);
  if (dep_mask & (1u << dim))
    return fail(SLDG_ERR_ARG, "dep_mask 0x%x contains the swept dimension %d", dep_mask, dim);
  if (!shift) return fail(SLDG_ERR_ARG, "null shift pointer");
  if (p->n_lo > 0 && (!in_lo || !out_lo)) return fail(SLDG_ERR_ARG, "null FP64-mode (mass) pointer");
  if (p->n_hi > 0 && (!in_hi || !out_hi)) return fail(SLDG_ERR_ARG, "null state (hi) pointer");
  const int64_t mb = p->lo_bytes, hb = p->hi_bytes;
  const void* ins[2] = {in_lo, in_hi};
  const int64_t insz[2] = {mb, hb};
  const void* outs[2] = {out_lo, out_hi};
  const int64_t outsz[2] = {mb, hb};
  for (int i = 0; i < 2; ++i)
    for (int o = 0; o < 2; ++o)
      if (insz[i] > 0 && outsz[o] > 0 && overlap(ins[i], insz[i], outs[o], outsz[o]))
        return fail(SLDG_ERR_ALIAS, "output buffer overlaps an input buffer");
  if (mb > 0 && hb > 0 && overlap(out_lo, mb, out_hi, hb))
    return fail(SLDG_ERR_ALIAS, "out_mass overlaps out_hi");
  int64_t sb = 8;
  for (int e = 0; e < p->ndim; ++e)
    if (dep_mask & (1u << e)) sb *= p->n[e];
  if ((mb > 0 && overlap(shift, sb, out_lo, mb)) || (hb > 0 && overlap(shift, sb, out_hi, hb)))
    return fail(SLDG_ERR_ALIAS, "shift overlaps an output buffer");
  return SLDG_OK;
}

// Describe the sweep along dim for the kernels (everything but the buffers).
void describe(const sldg_plan_s* p, int dim, uint32_t dep_mask, SweepArgs& a, int64_t& ntab) {
  describe_grid(p->ndim, p->n, p->o, p->modes, dim, dep_mask, p->rows_d[dim], p->tuples_d[dim],
                a, ntab);
  a.colwaves = dim > 0 ? (p->colwaves_d[dim] & 7) : 1;
}

// Whether the strided sweep described by `a` (with the plan's shape for its
// dimension) can run staged through LDS (sldg_staged.h): a narrow tier with
// at most the cell mean in FP64, 4 or 8 rows per thread, 1, 2 or 4 column
// waves, tiles of whole 64-column runs (P % (64 cw) == 0) and whole row
// chunks (N % ((4 / cw) L) == 0), 16-byte aligned planes, a tile within the
// LDS limit, and the planes of a tuple within 2^31 bytes (its buffer
// accesses take 32-bit byte offsets, with 2^31 as the out-of-range mark).
bool staged_fits(const sldg_plan_s* p, int dim, const SweepArgs& a, const void* in_hi,
                 const void* out_hi) {
  if (dim == 0 || a.lane || p->tier == SLDG_TIER_FP64 || p->ndouble > 1 || p->n_lo > 1) return false;
  const int L = a.chunk, cw = a.colwaves;
  if (!(L == 4 || L == 8) || !(cw == 1 || cw == 2 || cw == 4)) return false;
  if (a.P % (64 * cw) != 0 || a.N % ((4 / cw) * L) != 0) return false;
  if (((uintptr_t)in_hi | (uintptr_t)out_hi) & 15) return false;
  const int64_t sz = elem_size(p->tier);
  if (staged_lds_bytes(p->k, (int)sz, L, cw) > kStagedLdsMax) return false;
  return ((int64_t)(p->o - 1) * a.mstride + 1) * a.cells * sz <= (int64_t)INT32_MAX;
}

// Launch shapes the tuner tries: (rows, tuples, column waves).  Dimension-0
// sweeps use the tuple count, and rows to pick the group (4) or lane (1)
// form where the window form does not apply; strided sweeps with rows 0 run
// in the lane form.
constexpr int kTuneContig[][3] = {{4, 1, 1}, {4, 3, 1}, {4, 9, 1}, {4, 27, 1}, {4, 0, 1},
                                  {1, 1, 1}, {1, 3, 1}, {1, 9, 1}, {1, 27, 1}, {1, 0, 1}};
// Column waves 1, 2 or 4, with or without the staging and memory-order flags.
constexpr bool colwaves_valid(int c) {
  const int w = c & ~(SLDG_SHAPE_STAGED | SLDG_SHAPE_MEMORDER);
  return w == 1 || w == 2 || w == 4;
}

constexpr int kTuneStrided[][3] = {
    {2, 1, 1},  {2, 1, 2},  {2, 1, 4},  {2, 3, 1},  {2, 3, 2},  {2, 3, 4},  {2, 9, 1},
    {2, 9, 2},  {2, 9, 4},  {2, 27, 1}, {2, 27, 2}, {2, 27, 4}, {4, 1, 1},  {4, 1, 2},
    {4, 1, 4},  {4, 3, 1},  {4, 3, 2},  {4, 3, 4},  {4, 9, 1},  {4, 9, 2},  {4, 9, 4},
    {4, 27, 1}, {4, 27, 2}, {4, 27, 4}, {8, 1, 1},  {8, 1, 2},  {8, 1, 4},  {8, 3, 1},
    {8, 3, 2},  {8, 3, 4},  {8, 9, 1},  {8, 9, 2},  {8, 9, 4},  {8, 27, 1}, {8, 27, 2},
    {8, 27, 4}, {0, 1, 1},  {0, 3, 1},  {0, 9, 1},  {0, 27, 1}, {0, 0, 1},
    // staged through LDS (column waves + SLDG_SHAPE_STAGED)
    {4, 3, 17}, {4, 9, 17}, {4, 27, 17}, {4, 3, 18}, {4, 9, 18}, {4, 27, 18},
    {8, 3, 17}, {8, 9, 17}, {8, 27, 17}, {8, 3, 18}, {8, 9, 18}, {8, 27, 18},
    {4, 9, 20}, {4, 27, 20}, {8, 9, 20}, {8, 27, 20},
    // tiles in memory order (+ SLDG_SHAPE_MEMORDER), direct and staged
    {4, 3, 36}, {4, 9, 36}, {8, 3, 34}, {8, 9, 34}, {8, 3, 36}, {8, 9, 36},
    {4, 27, 50}, {4, 27, 52}, {8, 9, 50}, {8, 9, 52}};
constexpr int kNumTuneContig = sizeof(kTuneContig) / sizeof(kTuneContig[0]);
constexpr int kNumTuneStrided = sizeof(kTuneStrided) / sizeof(kTuneStrided[0]);


void free_plan(sldg_plan_s* p) {
  if (!p) return;
  for (int q = 0; q < p->nev_created; ++q) (void)hipEventDestroy(p->ev[q]);
  if (p->d_s) dev_free(p->d_s);
  if (p->d_ab) dev_free(p->d_ab);
  if (p->d_mass_part) dev_free(p->d_mass_part);
  if (p->d_mass_out) dev_free(p->d_mass_out);
  if (p->d_pmap) dev_free(p->d_pmap);
  if (p->d_hmode) dev_free(p->d_hmode);
  if (p->d_redo) dev_free(p->d_redo);
  if (p->d_part) dev_free(p->d_part);
  if (p->d_field) dev_free(p->d_field);
  if (p->h_mass_out) (void)hipHostFree(p->h_mass_out);
  delete p;
}

// Looks up, once per device, the address of that device's copy of the static
// field scratch (the device must be current).  Devices past kMaxDevices keep
// no address; the allocation-free entry point then reports it.
sldg_status scratch_setup(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return SLDG_OK;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev]) return SLDG_OK;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    (void)hipGetLastError();
    return device_error(e != hipSuccess ? e : hipErrorInvalidSymbol,
                        "hipGetSymbolAddress of the static field scratch");
  }
  g_scratch_ptr[dev] = static_cast<double*>(ptr);
  return SLDG_OK;
}

// The absmax partial buffer holds at least n floats (grown with dev_malloc;
// freeing the old one waits for the device).  It owns d_part alone: the
// field scratch is grown and freed only by ensure_field and free_plan.
sldg_status ensure_part(sldg_plan_s* p, int64_t n) {
  if (n <= p->part_cap) return SLDG_OK;
  if (p->d_part) dev_free(p->d_part);
  p->d_part = nullptr;
  p->part_cap = 0;
  hipError_t e = dev_malloc(&p->d_part, sizeof(float) * (size_t)n);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return e == hipErrorOutOfMemory ? fail(SLDG_ERR_NOMEM, "absmax partials: %s", hipGetErrorString(e))
                                    : device_error(e, "absmax partials");
  }
  p->part_cap = n;
  return SLDG_OK;
}

// Scale block views: int32 exp[n_hi], then float amax[n_hi].
struct ScaleBlock {
  int32_t* exp;
  float* amax;
};
ScaleBlock scale_view(const sldg_plan_s* p, const void* blk) {
  int32_t* e = static_cast<int32_t*>(const_cast<void*>(blk));
  return {e, reinterpret_cast<float*>(e + p->n_hi)};
}

sldg_status check_scaled(const sldg_plan_s* p, const void* in_scale, const void* out_scale,
                         const void* const* bufs, const int64_t* sizes, int nbuf) {
  if (p->tier != SLDG_TIER_FP16)
    return fail(SLDG_ERR_UNSUPPORTED, "scaled storage needs an FP16-tier plan");
  if (!in_scale || !out_scale) return fail(SLDG_ERR_ARG, "null scale block");
  const int64_t sb = 8 * p->n_hi;
  if (((uintptr_t)in_scale | (uintptr_t)out_scale) & 3)
    return fail(SLDG_ERR_ARG, "scale blocks must be 4-byte aligned");
  if (sb > 0 && overlap(in_scale, sb, out_scale, sb))
    return fail(SLDG_ERR_ALIAS, "input and output scale blocks overlap");
  for (int i = 0; i < nbuf; ++i)
    if (sb > 0 && sizes[i] > 0 && bufs[i] &&
        (overlap(out_scale, sb, bufs[i], sizes[i]) || overlap(in_scale, sb, bufs[i], sizes[i])))
      return fail(SLDG_ERR_ALIAS, "a scale block overlaps a state buffer");
  return SLDG_OK;
}

// Kernel timing: an event before and after a sweep launch (the line-table
// launch stays outside); `code` is the swept dimension, or kXYTimingDim for
// the fused pair.
sldg_status timing_begin(sldg_plan_s* p, bool& timed) {
  timed = p->timing && p->ntimed < kMaxTimed;
  if (!timed) return SLDG_OK;
  const int i = p->ntimed;
  if (2 * i + 1 >= p->nev_created) {
    for (int q = p->nev_created; q < 2 * i + 2; ++q) {
      hipError_t e = hipEventCreate(&p->ev[q]);
      if (e != hipSuccess) return device_error(e, "hipEventCreate");
      p->nev_created = q + 1;
    }
  }
  hipError_t e = hipEventRecord(p->ev[2 * i], p->stream);
  if (e != hipSuccess) return device_error(e, "hipEventRecord");
  return SLDG_OK;
}

sldg_status timing_end(sldg_plan_s* p, bool timed, int code) {
  if (!timed) return SLDG_OK;
  const int i = p->ntimed;
  hipError_t e = hipEventRecord(p->ev[2 * i + 1], p->stream);
  if (e != hipSuccess) return device_error(e, "hipEventRecord");
  p->ev_dim[i] = code;
  p->ntimed = i + 1;
  return SLDG_OK;
}

// Memory-order tiles of a strided sweep (strided_tile, SLDG_SHAPE_MEMORDER):
// where the column blocks of a workgroup tile the P columns of a slab
// exactly.  The XCD runs keep a column block's two row chunk groups, which
// share a halo row, on one XCD: with nblk blocks per group, the same block of
// the next group comes nblk tiles later, 16 or 8 runs of nblk / 16 or
// nblk / 8 tiles; other block counts take the dispatch order.  Measured on
// the 48^4 v2 sweep (P = 48^3, FP32-mode, 8 rows, 4 column waves): 0.638 ms
// in memory order with runs of 27, against 0.665 ms with the row chunk
// groups of a block together.
void set_memory_order(const sldg_plan_s* p, int dim, SweepArgs& a) {
  if (!(p->colwaves_d[dim] & SLDG_SHAPE_MEMORDER)) return;
  const int32_t cols = 64 * a.colwaves;
  if (a.P % cols != 0) return;
  a.nblk = a.P / cols;
  a.xcd = a.nblk % 16 == 0 ? a.nblk / 16 : a.nblk % 8 == 0 ? a.nblk / 8 : 0;
}

// One sweep.  With `pre` (a table offset into the plan's tables, entries
// first), its line tables were computed beforehand (split steps compute
// the tables of a whole sequence in one launch); otherwise they are computed
// here.
sldg_status run_sweep(sldg_plan_s* p, int dim, const double* shift, uint32_t dep_mask,
                      const double* in_lo, const void* in_hi, double* out_lo, void* out_hi,
                      bool adjoint = false, const void* in_scale = nullptr,
                      void* out_scale = nullptr, int64_t pre = -1) {
  SweepArgs a{};
  int64_t ntab = 0;
  describe(p, dim, dep_mask, a, ntab);
  a.xcd = dim == 0 ? p->xcd_contig : p->xcd_strided;
  if (dim > 0 && !a.lane) set_memory_order(p, dim, a);
  const bool scaled = in_scale != nullptr;
  ScaleBlock sin{}, sout{};
  if (scaled) {
    const int64_t nslot = sweep_slots(dim, a);
    // the kernels address the partials with 32-bit byte offsets
    if (nslot < 0 || nslot > INT32_MAX || p->n_hi * nslot > INT32_MAX / 4)
      return fail(SLDG_ERR_UNSUPPORTED, "sweep along dim %d: grid too large for one launch", dim);
    sldg_status st = ensure_part(p, std::max<int64_t>(1, p->n_hi * nslot));
    if (st != SLDG_OK) return st;
    sin = scale_view(p, in_scale);
    sout = scale_view(p, out_scale);
    a.in_exp = sin.exp;
    a.out_exp = sout.exp;
    a.amax_part = p->d_part;
    a.nslot = (int32_t)nslot;
  }
  if (ntab > p->table_cap)
    return fail(SLDG_ERR_ARG, "line table of %lld entries exceeds the plan's %lld",
                (long long)ntab, (long long)p->table_cap);
  const int64_t o2 = (int64_t)p->o * p->o;
  const int64_t toff = pre >= 0 ? pre : 0;
  hipError_t e = hipSuccess;
  if (pre < 0) {
    e = launch_line_tables(p->k, ntab, p->n[dim], shift, p->d_s, p->d_ab, true, adjoint,
                           p->stream);
    if (e != hipSuccess) return device_error(e, "line-table launch");
  }
  a.in_lo = in_lo;
  a.in_hi = in_hi;
  a.out_lo = out_lo;
  a.out_hi = out_hi;
  a.pmap = p->d_pmap;
  a.n_lo = (int32_t)p->n_lo;
  a.wide_fp64 = p->ndouble > 1 ? 1 : 0;
  a.s_tab = p->d_s + toff;
  a.ab_tab = p->d_ab + 2 * o2 * toff;
  a.ab_cs = ntab;
  a.stage = (p->colwaves_d[dim] & SLDG_SHAPE_STAGED) && staged_fits(p, dim, a, in_hi, out_hi) ? 1 : 0;
  bool timed = false;
  sldg_status tst = timing_begin(p, timed);
  if (tst != SLDG_OK) return tst;
  if (scaled) {
    e = launch_scale_predict(p->n_hi, sin.exp, sin.amax, sout.exp, p->scale_headroom, p->d_part,
                             p->n_hi * (int64_t)a.nslot, p->d_redo + p->n_hi, p->stream);
    if (e != hipSuccess) return device_error(e, "scale prediction launch");
  }
  e = launch_sweep(p->k, (int)p->tier, dim, a, p->stream);
  if (e == hipErrorInvalidConfiguration)
    return fail(SLDG_ERR_UNSUPPORTED, "sweep along dim %d: grid too large for one launch", dim);
  if (e != hipSuccess) return device_error(e, "sweep launch");
  if (scaled) {
    e = launch_scale_decide(p->n_hi, p->d_part, a.nslot, sout.exp, sout.amax, p->d_redo,
                            p->d_redo + p->n_hi,
                            p->stream);
    if (e != hipSuccess) return device_error(e, "scale decision launch");
    e = launch_scale_redo(p->k, dim, a, p->n_hi, p->d_redo, p->d_redo + p->n_hi, p->d_hmode,
                          p->stream);
    if (e != hipSuccess) return device_error(e, "scale repair launch");
  }
  return timing_end(p, timed, dim);
}

// The fused pair of sweeps along dimensions 0 and 1 (sldg_fused.h): the
// tile rows R of dimension 1 that fit the LDS budget and the phase-2 item
// limit, 0 if none does.  The budget keeps four workgroups per CU (160 KB of
// LDS): on the 48^4 workload taller tiles with fewer workgroups per CU
// measured slower in every tier (FP32: R = 24 at 3 per CU 0.81 ms, R = 16 at
// 4 per CU 0.64 ms).
constexpr int64_t kXYLdsBudget = 40 * 1024;
int32_t xy_tile_rows(const sldg_plan_s* p) {
  const int64_t N0 = p->n[0], N1 = p->n[1];
  static const int kCand[] = {48, 32, 24, 16, 12, 8, 6, 4, 3, 2, 1};
  for (int R : kCand) {
    if (p->xy_rows > 0 && R != p->xy_rows) continue;
    if (R > N1 && R > 1) continue;
    if (xy_lds_bytes(p->k, (int)elem_size(p->tier), (int32_t)N0, R) > kXYLdsBudget) continue;
    if ((int64_t)p->o * (R + 1) * (N0 / 4) > (int64_t)kXYMaxItems * 256) continue;
    // the same number of tiles, of equal height (N1 = 32: two of 16 rows and
    // not 24 + 8)
    const int64_t chunks = (N1 + R - 1) / R;
    return (int32_t)((N1 + chunks - 1) / chunks);
  }
  return 0;
}

// Whether the pair can run fused: the displacements of both sweeps are
// uniform over every (dimension 0, dimension 1) slab, at most the cell mean is
// FP64, rows of dimension 0 are whole 4-cell blocks, the buffers are 16-byte
// aligned and a tile fits.  Sets *why on refusal.
bool xy_eligible(const sldg_plan_s* p, uint32_t mask0, uint32_t mask1, const double* in_lo,
                 const void* in_hi, const double* out_lo, const void* out_hi, const char** why) {
  *why = nullptr;
  if (p->ndim < 2) *why = "needs two or more dimensions";
  else if ((mask0 | mask1) & 3u) *why = "a displacement depends on dimension 0 or 1";
  else if (p->n_lo > 1) *why = "more modes than the cell mean are FP64";
  else if (p->n[0] % 4) *why = "ncells[0] is not a multiple of 4";
  else if (((uintptr_t)in_hi | (uintptr_t)out_hi |
            (p->n_lo ? ((uintptr_t)in_lo | (uintptr_t)out_lo) : 0)) & 15)
    *why = "buffers not 16-byte aligned";
  else if (xy_tile_rows(p) == 0) *why = "a tile of the (0, 1) slab does not fit in LDS";
  else if (p->cells / (p->n[0] * p->n[1]) * (p->modes / (p->o * p->o)) *
               ((p->n[1] + xy_tile_rows(p) - 1) / xy_tile_rows(p)) > INT32_MAX)
    *why = "too many tiles for one launch";
  return *why == nullptr;
}

// The fused (0, 1) pair.  With pre0 >= 0 the two sweeps' tables were
// computed beforehand, at entries pre0 and pre1 of the plan's tables.
sldg_status run_xy(sldg_plan_s* p, const double* shift0, uint32_t mask0, const double* shift1,
                   uint32_t mask1, const double* in_lo, const void* in_hi, double* out_lo,
                   void* out_hi, int64_t pre0 = -1, int64_t pre1 = -1) {
  SweepArgs a0{}, a1{};
  int64_t nt0 = 0, nt1 = 0;
  describe(p, 0, mask0, a0, nt0);
  describe(p, 1, mask1, a1, nt1);
  if (nt0 + nt1 > p->table_cap)
    return fail(SLDG_ERR_UNSUPPORTED, "fused sweeps: line tables of %lld + %lld entries exceed %lld",
                (long long)nt0, (long long)nt1, (long long)p->table_cap);
  const int64_t o2 = (int64_t)p->o * p->o;
  hipError_t e = hipSuccess;
  if (pre0 < 0) {
    pre0 = 0;
    pre1 = nt0;
    e = launch_line_tables(p->k, nt0, p->n[0], shift0, p->d_s, p->d_ab, true, false, p->stream);
    if (e == hipSuccess)
      e = launch_line_tables(p->k, nt1, p->n[1], shift1, p->d_s + nt0, p->d_ab + 2 * o2 * nt0,
                             true, false, p->stream);
    if (e != hipSuccess) return device_error(e, "line-table launch");
  }
  const int32_t R = xy_tile_rows(p);
  XYArgs x{};
  x.in_lo = in_lo;
  x.in_hi = in_hi;
  x.out_lo = out_lo;
  x.out_hi = out_hi;
  x.n_lo = (int32_t)p->n_lo;
  x.cells = p->cells;
  x.N0 = (int32_t)p->n[0];
  x.N1 = (int32_t)p->n[1];
  x.Q = (int32_t)(p->cells / (p->n[0] * p->n[1]));
  x.R = R;
  x.nrc = (x.N1 + R - 1) / R;
  x.tstride = (int32_t)xy_tile_stride(x.N0, R);
  x.xcd = p->xcd_xy;
  x.one = 1.0f;
  x.fnb = FastDiv::make((uint32_t)(x.N0 / 4));
  x.fnrc = FastDiv::make((uint32_t)x.nrc);
  x.fQ = FastDiv::make((uint32_t)x.Q);
  x.s0 = p->d_s + pre0;
  x.ab0 = p->d_ab + 2 * o2 * pre0;
  x.cs0 = nt0;
  x.map0 = a0.map;
  x.s1 = p->d_s + pre1;
  x.ab1 = p->d_ab + 2 * o2 * pre1;
  x.cs1 = nt1;
  x.map1 = a1.map;
  const int64_t nblocks = (int64_t)x.nrc * x.Q * (p->modes / o2);
  bool timed = false;
  sldg_status tst = timing_begin(p, timed);
  if (tst != SLDG_OK) return tst;
  e = launch_xy(p->k, (int)p->tier, x, xy_lds_bytes(p->k, (int)elem_size(p->tier), x.N0, R),
                (int32_t)nblocks, p->stream);
  if (e != hipSuccess) return device_error(e, "fused sweep launch");
  return timing_end(p, timed, kXYTimingDim);
}

// Rows per wave of the X V X pass: a wave loads four rows more than it has and
// X-sweeps three more, but its rows follow one another, so the most (of 8, 4, 2, 1)
// that leaves kStrangWaves waves (of the chip's 1,024 SIMDs) where the grid is
// small.  Measured (five Strang
// steps, FP32-mode, rows 1, 2, 4, 8, 16): 256^2 k = 2 (1,280 wave rows) 49, 46,
// 53, 66, 99 us; 512^2 k = 3 (4,608) 138, 126, 123, 136, 204; 1024^2 k = 3
// (17,408) 351, 275, 251, 245, 285; 2048^2 k = 3 (69,632) 1414, 1085, 931, 864,
// 884.
constexpr int64_t kStrangWaves = 600;
constexpr int32_t kStrangRows = 8;

// Whether X V X (sweeps along dimensions 0, 1, 0) can run as one pass
// (sldg_strang.h): at most the cell mean FP64, a spectator group's planes
// below 2^31 bytes and a launchable grid.  Kernel timing measures the sweeps
// one by one, so it keeps them apart.
// The displacements are on the device, so the rule cannot see them.  Waves of
// spread V shifts walk each lane's own rows, which on (x, v) grids costs less than
// the sweeps (512^2, k = 2, FP32: 13 us a step with V shifts to 1.5 cells, 18 to 10,
// 25 to 30; the sweeps 24) but at k = 3 and 30 cells (42 us against 35).  On
// full-chip grids of three and more dimensions with short lines it can cost more:
// 64 x 200 x 32, shifts to 5 cells, k = 2, FP32 96 us against 73, k = 3, BF16 146
// against 105 (36 against 66 and 84 against 96 below one cell); sldg_plan_set_fusion
// turns the pass off.
bool strang_eligible(const sldg_plan_s* p, StrangArgs& x, int64_t& nblocks) {
  if (!p->fuse || p->timing || p->ndim < 2 || p->n_lo > 1) return false;
  const int64_t N0 = p->n[0], N1 = p->n[1];
  if (!strang_fits(p->cells, p->o, elem_size(p->tier))) return false;
  x.N0 = (int32_t)N0;
  x.N1 = (int32_t)N1;
  x.Q = (int32_t)(p->cells / (N0 * N1));
  const int64_t groups = p->modes / (p->o * p->o);
  const int64_t lines = (N0 + 61) / 62 * x.Q * groups * N1;    // wave rows
  if (!strang_pays(p->k, elem_size(p->tier), N0, lines)) return false;
  int32_t rows = kStrangRows;
  while (rows > 1 && lines / rows < kStrangWaves) rows >>= 1;
  strang_tiles(x, rows);
  nblocks = (int64_t)x.ntile * x.nstrip * x.Q * groups;
  return nblocks <= INT32_MAX;
}

// One X V X pass (post 1), or V X X with one X table (post 2, the first entry
// of mask and pre unused); the tables of the sweeps are at entries pre[i] of
// the plan's tables, those along dimension 0 entry-major.
sldg_status run_strang(sldg_plan_s* p, int post, const uint32_t (&mask)[3],
                       const int64_t (&pre)[3], const double* in_lo, const void* in_hi,
                       double* out_lo, void* out_hi) {
  StrangArgs x{};
  int64_t nblocks = 0;
  if (!strang_eligible(p, x, nblocks)) return fail(SLDG_ERR_UNSUPPORTED, "fused X V X sweeps");
  const int64_t E = 2LL * p->o * p->o;
  LineTable* tab[3] = {&x.x0, &x.v, &x.x1};
  for (int i = post == 2 ? 1 : 0; i < 3; ++i) {
    SweepArgs a{};
    int64_t nt = 0;
    describe(p, i == 1 ? 1 : 0, mask[i], a, nt);
    *tab[i] = {p->d_s + pre[i], p->d_ab + E * pre[i], i == 1 ? nt : 1, i == 1 ? 1 : E,
               (int32_t)(mask[i] >> (i == 1 ? 0 : 1) & 1), a.map};
  }
  x.in_lo = in_lo;
  x.in_hi = in_hi;
  x.out_lo = out_lo;
  x.out_hi = out_hi;
  x.n_lo = (int32_t)p->n_lo;
  x.cells = p->cells;
  x.xcd = p->xcd_strang;
  x.one = 1.0f;
  x.fstrip = FastDiv::make((uint32_t)x.nstrip);
  x.ftile = FastDiv::make((uint32_t)x.ntile);
  x.fQ = FastDiv::make((uint32_t)x.Q);
  const hipError_t e = launch_strang(p->k, (int)p->tier, post, x, (int32_t)nblocks, p->stream);
  if (e != hipSuccess) return device_error(e, "fused X V X launch");
  return SLDG_OK;
}

// Whether the sweeps along d >= 1 and d + 1 can run as one pass
// (sldg_colpair.h): displacements of the dimensions below d alone, at most the
// cell mean FP64, a plane within 31-bit byte offsets and a launchable grid; and
// whether it pays.  That takes three quarters of the lanes (columns below d
// over a whole number of waves: 48 of 64 columns x 160^2, k = 2, bf16: 65 us
// against 74 for the two sweeps; 40 columns 62 against 57, 16 columns 61 against
// 26), and four rows of d + 1 (a strip reads two more than it writes; 8192
// columns x 64 x 4 rows 270 us against 316, x 2 rows 207 against 172).  For
// k = 3 eight rows and seven eighths of the lanes: its waves hold one row of d
// and read three (12^4 cells, 144 columns in 192 lanes, FP64: 50 us against 36;
// 16^4 79 against 127).  Where the columns are no multiple of 16, the rows of a
// wave straddle cache lines, and the two sweeps read them faster as long as they
// find the state in the caches: from 16 to 128 MB a state the pair took 1.0 to 1.4
// times the sweeps over random grids (2938 x 2 x 74, k = 3, bf16, 58 MB: 85 us
// against 62; 37 x 99 x 10 x 7, k = 2, FP32, 82 against 62), below 0.5 to 0.7 (the
// launches) and above, where the two buffers leave the 256 MB cache, 0.6 to 0.8;
// aligned 0.8 in between.
// Sets everything but the buffers and tables.
bool colpair_eligible(const sldg_plan_s* p, int d, uint32_t mask1, uint32_t mask2, ColPairArgs& x,
                      int64_t& nblocks) {
  if (!p->fuse || d < 1 || d + 1 >= p->ndim || ((mask1 | mask2) >> d) || p->n_lo > 1) return false;
  if (p->cells * 8 > (int64_t)INT32_MAX) return false;
  int64_t P = 1, ms = 1;
  for (int e = 0; e < d; ++e) {
    P *= p->n[e];
    ms *= p->o;
  }
  x.P = (int32_t)P;
  x.N1 = (int32_t)p->n[d];
  x.N2 = (int32_t)p->n[d + 1];
  x.Q = (int32_t)(p->cells / (P * p->n[d] * p->n[d + 1]));
  x.ms = (int32_t)ms;
  const int64_t groups = p->modes / (p->o * p->o);
  x.nblk = (int32_t)((P + 63) / 64);
  const bool high = p->k == 3;
  if (x.N1 < 2 || x.N2 < (high ? 8 : 4) || P * 8 < (high ? 7 : 6) * 64LL * x.nblk) return false;
  const int64_t bytes = p->lo_bytes + p->hi_bytes;
  if (P % 16 && bytes > (16 << 20) && bytes <= (128 << 20)) return false;
  const int32_t L = colpair_rows(p->k, (int)p->tier);
  x.nrow = (x.N1 + L - 1) / L;
  const int64_t tiles = (int64_t)x.nblk * x.Q * groups;
  const int32_t whole = x.nrow % 4 == 0 ? 1 : x.nrow % 2 == 0 ? 2 : 4;
  // Workgroups of strips of R rows.
  auto workgroups = [&](int32_t R) {
    x.R = R;
    x.nstrip = (x.N2 + R - 1) / R;
    x.S = std::min(whole, x.nstrip);
    x.ngroup = (x.nstrip + x.S - 1) / x.S;
    x.nchunk = (x.nrow * x.S + 3) / 4;
    return tiles * x.ngroup * x.nchunk;
  };
  // Rows of d + 1 per wave: the least time, taken as the rows of a wave (R + 2, and
  // the tables for about one) times the rounds of workgroups on 256 compute units.  A
  // second workgroup on a unit takes 0.4 of the first's time more, and from there on
  // the time grows with the workgroups (fits of 699 random grids: 1.3 to 1.7 times the
  // first for two, 0.8 to 1.1 for each of many).  16^4, k = 2, FP32: 6 rows 25 us, 16
  // rows 33; 48^4: FP32 24 rows 727 us, 48 rows 749, bf16 448 and 433, k = 1 154 and
  // 165, hence the most rows.
  const int64_t most = p->k > 1 && (p->tier == SLDG_TIER_BF16 || p->tier == SLDG_TIER_FP16) ? 48 : 24;
  double best = 1e300;
  int32_t R = 0;
  for (int64_t ns = (x.N2 + most - 1) / most; ns <= (x.N2 + 3) / 4; ++ns) {
    const int32_t rows = (int32_t)((x.N2 + ns - 1) / ns);
    const double u = (double)workgroups(rows) / 256.0;
    const double cost = (rows + 3) * (u <= 1.0 ? 1.0 : std::max(1.4, 0.8 * u));
    if (cost < best) {
      best = cost;
      R = rows;
    }
  }
  nblocks = workgroups(R);
  // lines of both dimensions that the sweeps one by one hold in LDS
  ColSweepArgs line{};
  int64_t lds = 0;
  line.P = x.P;
  line.N = std::max(x.N1, x.N2);
  return nblocks <= INT32_MAX && p->cells / 8 * (p->modes / p->o) <= INT32_MAX &&
         colsweep_tiles(line, (int)p->o, elem_size(p->tier), lds);
}

// Spread flags of the pairs of a call: in the last entries of the plan's shift
// table, past the call's tables (which leave room for them).
constexpr int64_t kPairFlags = kMaxTableSet / 2;
int32_t* pair_flag(const sldg_plan_s* p, int i) { return p->d_s + p->table_cap - 1 - i; }

// The mean span of the shifts of 64 columns (largest less smallest, + 1) from
// which a pair's sweeps run one by one: the fused pass then reads scattered rows.
// Pass and sweeps (the plan's own), us: 48^4, k = 2, FP32 at spans 2.4, 4.4, 7.5 and
// 14 806, 1324, 2030, 4977 and 1346, 1402, 1513, 1771; BF16 546, 898, 1326, 2800 and
// 732, 736, 744, 993; FP64 1519, 2088, 2848, 6070 and 2618, 2655, 2784, 3441; 24^4,
// k = 3, FP32 at 2.4, 4.8 and 8.1 259, 449, 926 and 320, 383, 413; 128 x 100^2, k = 2,
// FP32 at 5, 8 and 14 87, 122, 183 and 134, 141, 156.
constexpr float pair_span(int k, sldg_tier tier) {
  return tier == SLDG_TIER_FP64 ? 7.0f : k == 3 ? 4.0f : 4.5f;
}

// States up to which the fused pass runs at any displacements: they stay in the
// caches, where scattered rows cost less than the launches of a choice (64^3, k =
// 1, FP32, 10 MB: 15, 18 and 23 us at spans of 6, 10 and 18 against 21 for the
// sweeps, 27 by line sweeps; 16^4, k = 1 10 us instead of 14; 64^3, k = 2, 30 MB 40
// us at 6 and 49 at 10 against 37; 16^4, k = 2, BF16, 11 MB, 40 at 16 against 32).
constexpr int64_t kPairSmall = 10 << 20;
bool pair_decides(const sldg_plan_s* p) { return p->lo_bytes + p->hi_bytes > kPairSmall; }

// The decision of the pair along d and d + 1 with displacements shift1 and shift2,
// at flag i (none for small states).
PairSpread pair_decision(const sldg_plan_s* p, int d, const double* shift1, uint32_t mask1,
                         const double* shift2, uint32_t mask2, int i) {
  PairSpread x{};
  if (!pair_decides(p)) return x;
  const double* const shift[2] = {shift1, shift2};
  const uint32_t mask[2] = {mask1, mask2};
  int64_t P = 1;
  for (int e = 0; e < d; ++e) P *= p->n[e];
  for (int w = 0; w < 2; ++w) {
    int64_t run = 1, n = 1;
    for (int e = 0; e < d; ++e) {
      if (mask[w] >> e & 1) n *= p->n[e];
      else if (n == 1) run *= p->n[e];
    }
    x.sigma[w] = shift[w];
    x.run[w] = FastDiv::make((uint32_t)run);
    x.n[w] = FastDiv::make((uint32_t)n);
    x.N[w] = (double)p->n[d + w];
    x.rN[w] = 1.0 / x.N[w];
  }
  x.P = (int32_t)P;
  x.most = pair_span(p->k, p->tier);
  x.flag = pair_flag(p, i);
  return x;
}

// One of the pair's sweeps by itself, where the flag is set (in place where the
// buffers are the same).
sldg_status run_colsweep(sldg_plan_s* p, int dim, uint32_t mask, int64_t pre, const int32_t* flag,
                         const double* in_lo, const void* in_hi, double* out_lo, void* out_hi) {
  SweepArgs a{};
  ColSweepArgs x{};
  describe(p, dim, mask, a, x.cs);
  x.in_lo = in_lo;
  x.in_hi = in_hi;
  x.out_lo = out_lo;
  x.out_hi = out_hi;
  x.n_lo = (int32_t)p->n_lo;
  x.cells = p->cells;
  x.P = a.P;
  x.N = a.N;
  x.Q = a.Q;
  x.ms = a.mstride;
  int64_t lds = 0;
  colsweep_tiles(x, (int)p->o, elem_size(p->tier), lds);
  x.ntile = (a.P + (1 << x.logc) - 1) >> x.logc;
  x.items = x.ntile * a.Q * a.nspec;
  x.one = 1.0f;
  x.ftile = FastDiv::make((uint32_t)x.ntile);
  x.fQ = FastDiv::make((uint32_t)x.Q);
  x.s = p->d_s + pre;
  x.ab = p->d_ab + 2LL * p->o * p->o * pre;
  x.map = a.map;
  x.flag = flag;
  const int32_t nblocks = (int32_t)std::min<int64_t>(x.items, 256 * std::min<int64_t>(8, kColSweepLdsMax / lds));
  const hipError_t e = launch_colsweep(p->k, (int)p->tier, x, nblocks, (int32_t)lds, p->stream);
  return e == hipSuccess ? SLDG_OK : device_error(e, "line sweep launch");
}

// The pair along d and d + 1, its tables at entries pre1 and pre2 of the plan's
// tables: in one pass, or one sweep after the other through LDS lines where flag
// i says that the shifts are too spread (large states).  The displacements are on the device, so
// all three launches are issued and those not wanted leave at once.
sldg_status run_colpair(sldg_plan_s* p, int d, uint32_t mask1, uint32_t mask2, int64_t pre1,
                        int64_t pre2, int i, const double* in_lo, const void* in_hi,
                        double* out_lo, void* out_hi) {
  ColPairArgs x{};
  int64_t nblocks = 0;
  if (!colpair_eligible(p, d, mask1, mask2, x, nblocks))
    return fail(SLDG_ERR_UNSUPPORTED, "fused sweeps along dimensions %d and %d", d, d + 1);
  const int64_t E = 2LL * p->o * p->o;
  SweepArgs a1{}, a2{};
  describe(p, d, mask1, a1, x.cs1);
  describe(p, d + 1, mask2, a2, x.cs2);
  x.map1 = a1.map;
  x.map2 = a2.map;
  x.s1 = p->d_s + pre1;
  x.ab1 = p->d_ab + E * pre1;
  x.s2 = p->d_s + pre2;
  x.ab2 = p->d_ab + E * pre2;
  x.in_lo = in_lo;
  x.in_hi = in_hi;
  x.out_lo = out_lo;
  x.out_hi = out_hi;
  x.n_lo = (int32_t)p->n_lo;
  x.cells = p->cells;
  x.one = 1.0f;
  x.fblk = FastDiv::make((uint32_t)x.nblk);
  x.fgroup = FastDiv::make((uint32_t)x.ngroup);
  x.frow = FastDiv::make((uint32_t)x.nrow);
  x.fchunk = FastDiv::make((uint32_t)x.nchunk);
  x.fQ = FastDiv::make((uint32_t)x.Q);
  x.flag = pair_decides(p) ? pair_flag(p, i) : nullptr;
  bool timed = false;
  sldg_status st = timing_begin(p, timed);
  if (st != SLDG_OK) return st;
  const hipError_t e = launch_colpair(p->k, (int)p->tier, x, (int32_t)nblocks, p->stream);
  if (e != hipSuccess) return device_error(e, "fused sweep launch");
  if (x.flag) st = run_colsweep(p, d, mask1, pre1, x.flag, in_lo, in_hi, out_lo, out_hi);
  if (st == SLDG_OK && x.flag)
    st = run_colsweep(p, d + 1, mask2, pre2, x.flag, out_lo, out_hi, out_lo, out_hi);
  if (st != SLDG_OK) return st;
  return timing_end(p, timed, kPairTimingDim);
}

constexpr int32_t kLineLds = 160 * 1024;      // LDS of a compute unit
constexpr int64_t kLineSweeps = 1 << 14;      // sweeps of one launch (some 50 ms at most)

// Whether split steps of a 1D problem can run as launches of many sweeps
// (sldg_line.h): the line fits the LDS and 1024 lanes of four cells, at most
// the cell mean FP64, no timing of single sweeps.  Faster over the whole range:
// 300 sweeps, k = 2, FP64, of 16 cells 61 us against 1132 sweep by sweep, 4096
// cells 402 against 1264.
bool line_steps_eligible(const sldg_plan_s* p) {
  return p->fuse && !p->timing && p->ndim == 1 && p->n_lo <= 1 && p->n[0] <= 4096 &&
         p->n[0] * line_cell_bytes(p->o, p->n_lo, elem_size(p->tier)) <= kLineLds;
}

// `total` sweeps of the sequence whose tables are at entries pre[q] of the
// plan's tables, from buffer cur on; cur becomes the buffer of the result.
sldg_status run_line_steps(sldg_plan_s* p, const std::vector<int64_t>& pre, int nseq, int64_t total,
                           double* const (&m)[2], void* const (&h)[2], int& cur) {
  LineStepsArgs x{};
  x.n_lo = (int32_t)p->n_lo;
  x.N = (int32_t)p->n[0];
  x.nseq = nseq;
  x.one = 1.0f;
  x.s = p->d_s;
  x.ab = p->d_ab;
  for (int q = 0; q < nseq; ++q) x.pre[q] = (int32_t)pre[(size_t)q];
  const int32_t bytes =
      (int32_t)((x.N * line_cell_bytes(p->o, p->n_lo, elem_size(p->tier)) + 15) & ~15LL);
  x.stride = 2 * bytes <= kLineLds ? bytes : 0;
  // as many lanes as a workgroup holds: fewer lanes of more cells take longer
  // (256 cells, k = 2, FP64, 300 sweeps: 85, 109, 161 us at 1, 2, 4 cells a lane)
  const int cells = x.N <= 1024 ? 1 : x.N <= 2048 ? 2 : 4;
  // each launch starts at the first sweep of the sequence
  const int64_t most = std::max<int64_t>(kLineSweeps / nseq, 1) * nseq;
  for (int64_t done = 0; done < total; done += x.sweeps) {
    x.sweeps = (int32_t)std::min(most, total - done);
    const int to = cur ^ (x.sweeps & 1);
    x.in_lo = m[cur];
    x.in_hi = h[cur];
    x.out_lo = m[to];
    x.out_hi = h[to];
    const hipError_t e = launch_line_steps(p->k, (int)p->tier, x, cells,
                                           x.stride ? 2 * x.stride : bytes, p->stream);
    if (e != hipSuccess) return device_error(e, "1D steps launch");
    cur = to;
  }
  return SLDG_OK;
}

// Default launch shape of a strided sweep (the tuner picks per dimension): 4 rows a
// thread, or 8 with 2 column waves, which read fewer halo rows, on grids of 3/4
// million cells of four dimensions on, along dimensions of 16 cells on whose last
// chunk of 8 rows is not much emptier than of 4 (for k = 1, whose sweeps are
// short, no emptier).  From 2^22 cells on staged for the 16-bit tiers.  Over 30
// grids of 4 to 6 dimensions and every degree and tier 8 rows under this rule take
// 0.87 (scaled FP16), 0.95 (BF16) and 0.96 (FP32, FP64) of the time of 4 rows, one
// sweep in a hundred 3-11% more; without it the same shape costs 1024 x 8 x 10 x 10,
// k = 3, BF16 350 us against 288 (10 rows in chunks of 8) and, staged, 64^3 x 3, k =
// 2, BF16 59 us against 48.  48^4, k = 2: scaled FP16 432-567 us a strided sweep
// against 646-671, BF16 356-431 against 413-477.  Smaller grids and fewer dimensions
// have too few waves (64^3, k = 2: 18-24 us against 13-16).
bool eight_rows(const sldg_plan_s* p, int d) {
  if (p->ndim < 4 || p->cells < 3 << 18 || p->n[d] < 16) return false;
  const int64_t pad4 = (p->n[d] + 3) / 4 * 4, pad8 = (p->n[d] + 7) / 8 * 8;
  return p->k == 1 ? pad8 <= pad4 : 7 * pad8 <= 8 * pad4;
}

}  // namespace

extern "C" {

sldg_status sldg_set_device_alloc_limit(int64_t bytes) {
  if (bytes < -1) return fail(SLDG_ERR_ARG, "allocation limit %lld < -1", (long long)bytes);
  std::lock_guard<std::mutex> lock(g_alloc_mu);
  g_alloc_limit = bytes;
  return ok();
}

int64_t sldg_device_alloc_bytes(void) {
  std::lock_guard<std::mutex> lock(g_alloc_mu);
  return g_alloc_live;
}

const char* sldg_status_string(sldg_status s) {
  switch (s) {
    case SLDG_OK: return "ok";
    case SLDG_ERR_ARG: return "invalid argument";
    case SLDG_ERR_ALIAS: return "output overlaps input";
    case SLDG_ERR_UNSUPPORTED: return "unsupported configuration";
    case SLDG_ERR_NOMEM: return "out of device memory";
    case SLDG_ERR_DEVICE: return "device error";
  }
  return "unknown status";
}

const char* sldg_last_error(void) { return last_error_text(); }

sldg_status sldg_plan(sldg_plan_t* out, int ndim, const int64_t* ncells, int k, sldg_tier tier,
                      void* stream) {
  return sldg_plan_ex(out, ndim, ncells, k, tier, 1, stream);
}

sldg_status sldg_plan_ex(sldg_plan_t* out, int ndim, const int64_t* ncells, int k,
                         sldg_tier tier, int ndouble, void* stream) {
  if (!out) return fail(SLDG_ERR_ARG, "plan out-pointer is NULL");
  *out = nullptr;
  if (ndim < 1 || ndim > kMaxDim) return fail(SLDG_ERR_ARG, "ndim %d not in [1, %d]", ndim, kMaxDim);
  if (!ncells) return fail(SLDG_ERR_ARG, "ncells is NULL");
  if (k < 1 || k > 3) return fail(SLDG_ERR_UNSUPPORTED, "degree k=%d not in [1, 3]", k);
  if ((int)tier < 0 || (int)tier > 3) return fail(SLDG_ERR_UNSUPPORTED, "tier %d unknown", (int)tier);
  if (ndouble < 0 || ndouble > ndim * k + 1)
    return fail(SLDG_ERR_ARG, "ndouble %d not in [0, %d]", ndouble, ndim * k + 1);
  int64_t cells = 1, min_n = INT64_MAX;
  for (int e = 0; e < ndim; ++e) {
    if (ncells[e] < 1) return fail(SLDG_ERR_ARG, "ncells[%d] = %lld < 1", e, (long long)ncells[e]);
    if (ncells[e] >= (1LL << 31))
      return fail(SLDG_ERR_UNSUPPORTED, "ncells[%d] too large", e);
    cells *= ncells[e];
    if (cells >= (1LL << 31))
      return fail(SLDG_ERR_UNSUPPORTED, "grid of >= 2^31 cells is not supported");
    min_n = std::min(min_n, ncells[e]);
  }
  sldg_plan_s* p = new (std::nothrow) sldg_plan_s{};
  if (!p) return fail(SLDG_ERR_NOMEM, "host allocation failed");
  p->ndim = ndim;
  for (int e = 0; e < ndim; ++e) p->n[e] = ncells[e];
  p->k = k;
  p->o = k + 1;
  p->tier = tier;
  p->stream = static_cast<hipStream_t>(stream);
  p->cells = cells;
  p->modes = 1;
  for (int e = 0; e < ndim; ++e) p->modes *= p->o;
  p->ndouble = ndouble;
  p->h_pmap.resize(p->modes);
  p->n_lo = p->n_hi = 0;
  for (int64_t m = 0; m < p->modes; ++m) {
    int deg = 0;
    for (int64_t r = m, e = 0; e < ndim; ++e, r /= p->o) deg += (int)(r % p->o);
    p->h_pmap[m] = deg < ndouble ? (int32_t)(-1 - p->n_lo++) : (int32_t)(p->n_hi++);
  }
  p->lo_bytes = p->n_lo * cells * 8;
  p->hi_bytes = p->n_hi * cells * elem_size(tier);
  // the most lines any sweep can have, and the (transverse cell, node) entries
  // of a collocated sweep
  int64_t max_n = 0;
  for (int e = 0; e < ndim; ++e) max_n = std::max<int64_t>(max_n, ncells[e]);
  p->table_cap = std::max<int64_t>(cells / min_n, (int64_t)(k + 1) * max_n);
  // launch shape of every dimension from the environment, if set
  int rows = 0, tuples = 9, colwaves = 0;
  p->xcd_contig = 8;           // run lengths measured best on MI355X (4D k = 2)
  p->xcd_strided = 16;
  p->fuse = 1;
  p->xy_rows = 0;
  p->xcd_xy = 0;               // the fused pass: dispatch order measured best
  p->xcd_strang = 16;          // 2048^2 k = 3 FP32-mode: 0.172 ms a pass, 0.174 at 8, 0.199 in dispatch order
  if (const char* env = getenv("SLDG_XY_ROWS")) p->xy_rows = std::max(0, atoi(env));
  if (const char* env = getenv("SLDG_XCD_XY")) p->xcd_xy = std::max(0, atoi(env));
  if (const char* env = getenv("SLDG_COLWAVES")) {
    const int c = atoi(env);
    if (colwaves_valid(c)) colwaves = c;
  }
  if (const char* env = getenv("SLDG_XCD_CONTIG")) p->xcd_contig = std::max(-1, atoi(env));
  if (const char* env = getenv("SLDG_XCD_STRIDED")) p->xcd_strided = std::max(-1, atoi(env));
  p->scale_headroom = 8;
  if (const char* env = getenv("SLDG_TUPLES")) {
    const int g = atoi(env);
    if (g >= 0) tuples = g;
  }
  if (const char* env = getenv("SLDG_STRIDED_ROWS")) {
    const int r = atoi(env);
    if (r == 1 || r == 2 || r == 4 || r == 8) rows = r;
  }
  for (int d = 0; d < kMaxDim; ++d) {
    const bool eight = d < ndim && eight_rows(p, d);
    const int stage = eight && elem_size(tier) == 2 && cells >= 1 << 22 ? SLDG_SHAPE_STAGED : 0;
    p->rows_d[d] = rows > 0 ? rows : eight ? 8 : 4;
    p->tuples_d[d] = tuples;
    p->colwaves_d[d] = colwaves > 0 ? colwaves : eight ? 2 | stage : 1;
  }
  p->rows_d[0] = 0;         // dimension 0: automatic form
  const int64_t o2 = (int64_t)p->o * p->o;
  p->mass_nblocks = mass_blocks(cells);
  // the plan's device tables, checked against the allocation limit before any
  // device call
  const int64_t plan_bytes = (int64_t)sizeof(int32_t) * p->table_cap +
                             (int64_t)sizeof(double) * 2 * o2 * p->table_cap +
                             (int64_t)sizeof(double) * (2 * p->mass_nblocks + 2) +
                             (int64_t)sizeof(int32_t) * p->modes +
                             (tier == SLDG_TIER_FP16 ? (int64_t)sizeof(int32_t) * 2 * p->n_hi : 0);
  if (!dev_alloc_fits(plan_bytes)) {
    free_plan(p);
    return fail(SLDG_ERR_NOMEM, "plan tables: %lld bytes exceed the device allocation limit",
                (long long)plan_bytes);
  }
  hipError_t e = hipGetDevice(&p->device);
  if (e != hipSuccess) {
    free_plan(p);
    return device_error(e, "hipGetDevice");
  }
  if (scratch_setup(p->device) != SLDG_OK) {
    free_plan(p);
    return SLDG_ERR_DEVICE;
  }
  e = dev_malloc(&p->d_s, sizeof(int32_t) * p->table_cap);
  if (e == hipSuccess) e = dev_malloc(&p->d_ab, sizeof(double) * 2 * o2 * p->table_cap);
  if (e == hipSuccess) e = dev_malloc(&p->d_mass_part, sizeof(double) * 2 * p->mass_nblocks);
  if (e == hipSuccess) e = dev_malloc(&p->d_mass_out, sizeof(double) * 2);
  if (e == hipSuccess) e = hipHostMalloc(&p->h_mass_out, sizeof(double) * 2, hipHostMallocDefault);
  if (e == hipSuccess) e = dev_malloc(&p->d_pmap, sizeof(int32_t) * p->modes);
  if (e == hipSuccess)
    e = hipMemcpy(p->d_pmap, p->h_pmap.data(), sizeof(int32_t) * p->modes, hipMemcpyHostToDevice);
  if (e == hipSuccess && tier == SLDG_TIER_FP16 && p->n_hi > 0) {
    std::vector<int32_t> hmode((size_t)p->n_hi);
    for (int64_t m = 0; m < p->modes; ++m)
      if (p->h_pmap[m] >= 0) hmode[(size_t)p->h_pmap[m]] = (int32_t)m;
    e = dev_malloc(&p->d_hmode, sizeof(int32_t) * p->n_hi);
    if (e == hipSuccess) e = dev_malloc(&p->d_redo, sizeof(int32_t) * (p->n_hi + 1));
    if (e == hipSuccess)
      e = hipMemcpy(p->d_hmode, hmode.data(), sizeof(int32_t) * p->n_hi, hipMemcpyHostToDevice);
  }
  if (e != hipSuccess) {
    const bool nomem = (e == hipErrorOutOfMemory);
    free_plan(p);
    (void)hipGetLastError();
    return nomem ? fail(SLDG_ERR_NOMEM, "plan tables: %s", hipGetErrorString(e))
                 : device_error(e, "plan tables");
  }
  *out = p;
  return ok();
}

void sldg_plan_destroy(sldg_plan_t p) {
  if (!p) return;
  (void)hipStreamSynchronize(p->stream);
  free_plan(p);
}

sldg_status sldg_plan_set_stream(sldg_plan_t p, void* stream) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  p->stream = static_cast<hipStream_t>(stream);
  return ok();
}

int64_t sldg_hi_bytes(sldg_plan_t p) { return p ? p->hi_bytes : -1; }

int64_t sldg_lo_planes(sldg_plan_t p) { return p ? p->n_lo : -1; }

int64_t sldg_hi_planes(sldg_plan_t p) { return p ? p->n_hi : -1; }

sldg_status sldg_plane_map(sldg_plan_t p, int32_t* out) {
  if (!p || !out) return fail(SLDG_ERR_ARG, "null pointer");
  std::copy(p->h_pmap.begin(), p->h_pmap.end(), out);
  return ok();
}

sldg_status sldg_timing_enable(sldg_plan_t p, int enable) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  p->timing = enable != 0;
  if (p->timing) p->ntimed = 0;
  return ok();
}

sldg_status sldg_timing_read(sldg_plan_t p, int dim, int64_t* launches, double* total_ms) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (!launches || !total_ms) return fail(SLDG_ERR_ARG, "null output pointer");
  if (dim < -3 || dim >= p->ndim) return fail(SLDG_ERR_ARG, "dim %d out of range", dim);
  hipError_t e = hipStreamSynchronize(p->stream);
  if (e != hipSuccess) return device_error(e, "hipStreamSynchronize");
  int64_t n = 0;
  double tot = 0.0;
  for (int i = 0; i < p->ntimed; ++i) {
    const int d = p->ev_dim[i];
    const bool match = (dim >= 0)    ? (d == dim)
                       : dim == -1   ? d == 0
                       : dim == -2   ? d > 0
                                     : d == kXYTimingDim;
    if (!match) continue;
    float ms = 0.f;
    e = hipEventElapsedTime(&ms, p->ev[2 * i], p->ev[2 * i + 1]);
    if (e != hipSuccess) return device_error(e, "hipEventElapsedTime");
    ++n;
    tot += ms;
  }
  *launches = n;
  *total_ms = tot;
  return ok();
}

sldg_status sldg_line_tables(sldg_plan_t p, int64_t n, int64_t period, const double* sigma,
                             int32_t* s_out, double* ab_out) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (n < 0 || period < 1) return fail(SLDG_ERR_ARG, "n=%lld period=%lld", (long long)n, (long long)period);
  if (n > 0 && (!sigma || !s_out || !ab_out)) return fail(SLDG_ERR_ARG, "null pointer");
  if (period >= (1LL << 31)) return fail(SLDG_ERR_ARG, "period too large");
  hipError_t e = launch_line_tables(p->k, n, period, sigma, s_out, ab_out, false, false,
                                    p->stream);
  if (e != hipSuccess) return device_error(e, "line-table launch");
  return ok();
}

sldg_status sldg_advect_dim(sldg_plan_t p, int dim, const double* shift, uint32_t dep_mask,
                            const double* in_mass, const void* in_hi, double* out_mass,
                            void* out_hi) {
  sldg_status st = check_sweep(p, dim, shift, dep_mask, in_mass, in_hi, out_mass, out_hi);
  if (st != SLDG_OK) return st;
  st = run_sweep(p, dim, shift, dep_mask, in_mass, in_hi, out_mass, out_hi);
  return st == SLDG_OK ? ok() : st;
}

sldg_status sldg_advect_dim_adjoint(sldg_plan_t p, int dim, const double* shift,
                                    uint32_t dep_mask, const double* in_mass, const void* in_hi,
                                    double* out_mass, void* out_hi) {
  sldg_status st = check_sweep(p, dim, shift, dep_mask, in_mass, in_hi, out_mass, out_hi);
  if (st != SLDG_OK) return st;
  st = run_sweep(p, dim, shift, dep_mask, in_mass, in_hi, out_mass, out_hi, true);
  return st == SLDG_OK ? ok() : st;
}

// nsteps times the sweeps of seq (adjoint: their transposes, in the order
// given).
static sldg_status run_steps(sldg_plan_t p, const sldg_sweep_desc* seq, int nseq, int nsteps,
                             bool adjoint, double* const (&m)[2], void* const (&h)[2],
                             int* result_buffer) {
  // validate every sweep against both directions before launching anything
  for (int q = 0; q < nseq; ++q) {
    for (int b = 0; b < 2; ++b) {
      sldg_status st = check_sweep(p, seq[q].dim, seq[q].shift, seq[q].dep_mask, m[b], h[b],
                                   m[1 - b], h[1 - b]);
      if (st != SLDG_OK) return st;
    }
  }
  // sweeps along dimension 0 then 1 run as one fused pass where they can
  // (same result, one read and one write of the state instead of two); the
  // pair's result then lands in the other buffer than two sweeps would leave
  // it in, which *result_buffer reports.  Elsewhere sweeps along 0, 1, 0 run
  // as one pass (three sweeps and one pass end in the same buffer).  Sweeps
  // along d >= 1 then d + 1 run as one where that pays; a caller that does not
  // ask for the result's buffer finds it where (0, 1) pairs alone leave it: the
  // last step then runs one such pair as two sweeps if need be.
  int pairs = 0;
  std::vector<char> fused((size_t)std::max(nseq, 1), 0);
  for (int q = 0; p->fuse && q + 1 < nseq; ++q) {
    const char* why = nullptr;
    StrangArgs x{};
    int64_t nblocks = 0;
    ColPairArgs cp{};
    if (seq[q].dim > 0 && seq[q + 1].dim == seq[q].dim + 1 &&
        colpair_eligible(p, seq[q].dim, seq[q].dep_mask, seq[q + 1].dep_mask, cp, nblocks)) {
      fused[(size_t)q] = 4;
      ++pairs;
      ++q;
      continue;
    }
    if (seq[q].dim != 0 || seq[q + 1].dim != 1) continue;
    if (!adjoint &&
        xy_eligible(p, seq[q].dep_mask, seq[q + 1].dep_mask, m[0], h[0], m[1], h[1], &why)) {
      fused[(size_t)q] = 2;
      ++q;
    } else if (q + 2 < nseq && seq[q + 2].dim == 0 && strang_eligible(p, x, nblocks)) {
      fused[(size_t)q] = 3;
      q += 2;
    }
  }
  // The line tables of every sweep of the sequence, in one launch before the
  // steps: the displacements are fixed over the call, so every step's tables
  // are these, and sweeps along the same dimension with the same displacements
  // and table layout share one.  Where the sequence's tables do not fit the
  // plan's table storage together, each sweep computes its own (and X V X runs
  // sweep by sweep).
  std::vector<int64_t> pre((size_t)std::max(nseq, 1), -1);
  std::vector<int> flag((size_t)std::max(nseq, 1), 0);
  if (nsteps > 0 && nseq > 0 && nseq <= kMaxTableSet) {
    TableSet set{};
    int64_t tot = 0;
    int of[kMaxTableSet];
    bool em[kMaxTableSet];
    for (int q = 0; q < nseq; ++q) {
      of[q] = -1;
      em[q] = fused[(size_t)q] == 3 || (q >= 2 && fused[(size_t)q - 2] == 3);
      for (int e = 0; e < q && of[q] < 0; ++e)
        if (seq[e].dim == seq[q].dim && seq[e].dep_mask == seq[q].dep_mask &&
            seq[e].shift == seq[q].shift && em[e] == em[q])
          of[q] = of[e];
      if (of[q] >= 0) continue;
      SweepArgs a{};
      int64_t nt = 0;
      describe(p, seq[q].dim, seq[q].dep_mask, a, nt);
      const int i = of[q] = set.count++;
      set.first[i] = tot;
      set.period[i] = p->n[seq[q].dim];
      set.sigma[i] = seq[q].shift;
      if (em[q]) set.entry_major |= 1u << i;
      if (adjoint) set.adjoint |= 1u << i;
      tot += nt;
    }
    set.first[set.count] = tot;
    if (pairs && tot + kPairFlags > p->table_cap) {
      for (char& f : fused) f = f == 4 ? 0 : f;
      pairs = 0;
    }
    if (tot <= p->table_cap) {
      // pairs with the same tables share a flag; the first is decided beside the
      // tables
      for (int q = 0, i = 0; q + 1 < nseq; ++q) {
        if (fused[(size_t)q] != 4) continue;
        int f = -1;
        for (int e = 0; e < q && f < 0; ++e)
          if (fused[(size_t)e] == 4 && of[e] == of[q] && of[e + 1] == of[q + 1]) f = flag[(size_t)e];
        if (f < 0) {
          f = i++;
          const PairSpread x = pair_decision(p, seq[q].dim, seq[q].shift, seq[q].dep_mask,
                                             seq[q + 1].shift, seq[q + 1].dep_mask, f);
          if (f == 0) set.pair = x;
          const hipError_t e = f > 0 && x.flag ? launch_pair_spread(x, p->stream) : hipSuccess;
          if (e != hipSuccess) return device_error(e, "pair decision launch");
        }
        flag[(size_t)q] = f;
      }
      const hipError_t e = launch_line_tables_set(p->k, set, p->d_s, p->d_ab, p->stream);
      if (e != hipSuccess) return device_error(e, "line-table launch");
      for (int q = 0; q < nseq; ++q) pre[(size_t)q] = set.first[of[q]];
    }
  }
  int cur = 0;
  if (pre[0] >= 0 && (int64_t)nseq * nsteps > 1 && line_steps_eligible(p)) {
    const sldg_status st = run_line_steps(p, pre, nseq, (int64_t)nseq * nsteps, m, h, cur);
    if (st != SLDG_OK) return st;
    if (result_buffer) *result_buffer = cur;
    return ok();
  }
  bool split = !result_buffer && (int64_t)pairs * nsteps % 2;
  for (int n = 0; n < nsteps; ++n) {
    for (int q = 0; q < nseq; ++q) {
      sldg_status st;
      if (split && n + 1 == nsteps && fused[(size_t)q] == 4) {
        fused[(size_t)q] = 0;
        split = false;
      }
      if (fused[(size_t)q] == 2) {
        st = run_xy(p, seq[q].shift, seq[q].dep_mask, seq[q + 1].shift, seq[q + 1].dep_mask,
                    m[cur], h[cur], m[1 - cur], h[1 - cur], pre[(size_t)q], pre[(size_t)q + 1]);
        ++q;
      } else if (fused[(size_t)q] == 3 && pre[(size_t)q] >= 0) {
        const uint32_t mask[3] = {seq[q].dep_mask, seq[q + 1].dep_mask, seq[q + 2].dep_mask};
        const int64_t at[3] = {pre[(size_t)q], pre[(size_t)q + 1], pre[(size_t)q + 2]};
        st = run_strang(p, 1, mask, at, m[cur], h[cur], m[1 - cur], h[1 - cur]);
        q += 2;
      } else if (fused[(size_t)q] == 4 && pre[(size_t)q] >= 0) {
        st = run_colpair(p, seq[q].dim, seq[q].dep_mask, seq[q + 1].dep_mask, pre[(size_t)q],
                         pre[(size_t)q + 1], flag[(size_t)q], m[cur], h[cur], m[1 - cur], h[1 - cur]);
        ++q;
      } else {
        st = run_sweep(p, seq[q].dim, seq[q].shift, seq[q].dep_mask, m[cur], h[cur], m[1 - cur],
                       h[1 - cur], adjoint, nullptr, nullptr, pre[(size_t)q]);
      }
      if (st != SLDG_OK) return st;
      cur = 1 - cur;
    }
  }
  if (result_buffer) *result_buffer = cur;
  return ok();
}

sldg_status sldg_split_steps(sldg_plan_t p, const sldg_sweep_desc* seq, int nseq, int nsteps,
                             double* mass0, void* hi0, double* mass1, void* hi1,
                             int* result_buffer) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (nseq < 0 || nsteps < 0 || (nseq > 0 && !seq))
    return fail(SLDG_ERR_ARG, "bad sweep sequence (nseq=%d nsteps=%d)", nseq, nsteps);
  double* const m[2] = {mass0, mass1};
  void* const h[2] = {hi0, hi1};
  return run_steps(p, seq, nseq, nsteps, false, m, h, result_buffer);
}

sldg_status sldg_split_steps_adjoint(sldg_plan_t p, const sldg_sweep_desc* seq, int nseq,
                                     int nsteps, double* mass0, void* hi0, double* mass1,
                                     void* hi1, int* result_buffer) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (nseq < 0 || nsteps < 0 || (nseq > 0 && !seq))
    return fail(SLDG_ERR_ARG, "bad sweep sequence (nseq=%d nsteps=%d)", nseq, nsteps);
  std::vector<sldg_sweep_desc> rev((size_t)nseq);
  for (int q = 0; q < nseq; ++q) rev[(size_t)q] = seq[nseq - 1 - q];
  double* const m[2] = {mass0, mass1};
  void* const h[2] = {hi0, hi1};
  return run_steps(p, rev.data(), nseq, nsteps, true, m, h, result_buffer);
}

sldg_status sldg_advect_dims01(sldg_plan_t p, const double* shift0, uint32_t dep_mask0,
                               const double* shift1, uint32_t dep_mask1, const double* in_mass,
                               const void* in_hi, double* out_mass, void* out_hi) {
  sldg_status st = check_sweep(p, 0, shift0, dep_mask0, in_mass, in_hi, out_mass, out_hi);
  if (st != SLDG_OK) return st;
  st = check_sweep(p, 1, shift1, dep_mask1, in_mass, in_hi, out_mass, out_hi);
  if (st != SLDG_OK) return st;
  const char* why = nullptr;
  if (!xy_eligible(p, dep_mask0, dep_mask1, in_mass, in_hi, out_mass, out_hi, &why))
    return fail(SLDG_ERR_UNSUPPORTED, "fused sweeps along dimensions 0 and 1: %s", why);
  st = run_xy(p, shift0, dep_mask0, shift1, dep_mask1, in_mass, in_hi, out_mass, out_hi);
  return st == SLDG_OK ? ok() : st;
}

sldg_status sldg_plan_set_fusion(sldg_plan_t p, int enable) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  p->fuse = enable != 0;
  return ok();
}

sldg_status sldg_plan_set_shape(sldg_plan_t p, int dim, int rows, int tuples, int colwaves) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (dim < 0 || dim >= p->ndim) return fail(SLDG_ERR_ARG, "dim %d out of range", dim);
  if (!(rows == 0 || rows == 1 || rows == 2 || rows == 4 || rows == 8))
    return fail(SLDG_ERR_ARG, "rows %d not in {0, 1, 2, 4, 8}", rows);
  if (tuples < 0) return fail(SLDG_ERR_ARG, "tuples %d < 0", tuples);
  if (!colwaves_valid(colwaves))
    return fail(SLDG_ERR_ARG, "colwaves %d: not 1, 2 or 4 plus SLDG_SHAPE_STAGED and "
                "SLDG_SHAPE_MEMORDER flags", colwaves);
  p->rows_d[dim] = rows;
  p->tuples_d[dim] = tuples;
  p->colwaves_d[dim] = colwaves;
  return ok();
}

sldg_status sldg_plan_get_shape(sldg_plan_t p, int dim, int* rows, int* tuples, int* colwaves) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (dim < 0 || dim >= p->ndim) return fail(SLDG_ERR_ARG, "dim %d out of range", dim);
  if (rows) *rows = p->rows_d[dim];
  if (tuples) *tuples = p->tuples_d[dim];
  if (colwaves) *colwaves = p->colwaves_d[dim];
  return ok();
}

sldg_status sldg_plan_sweep_form(sldg_plan_t p, int dim, uint32_t dep_mask, const double* in_lo,
                                 const void* in_hi, const double* out_lo, const void* out_hi,
                                 int* form) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (!form) return fail(SLDG_ERR_ARG, "form is NULL");
  if (dim < 0 || dim >= p->ndim) return fail(SLDG_ERR_ARG, "dim %d out of range", dim);
  if ((dep_mask >> p->ndim) || (dep_mask & (1u << dim)))
    return fail(SLDG_ERR_ARG, "dep_mask 0x%x invalid for dim %d", dep_mask, dim);
  SweepArgs a{};
  int64_t ntab = 0;
  describe(p, dim, dep_mask, a, ntab);
  a.in_lo = in_lo;
  a.in_hi = in_hi;
  a.out_lo = const_cast<double*>(out_lo);
  a.out_hi = const_cast<void*>(out_hi);
  a.n_lo = (int32_t)p->n_lo;
  a.wide_fp64 = p->ndouble > 1 ? 1 : 0;
  a.stage = (p->colwaves_d[dim] & SLDG_SHAPE_STAGED) && staged_fits(p, dim, a, in_hi, out_hi) ? 1 : 0;
  const int f = sweep_form(dim, a);
  if (f < 0) return fail(SLDG_ERR_UNSUPPORTED, "sweep along dim %d: grid too large", dim);
  *form = f;
  return ok();
}

sldg_status sldg_tune_candidate(int strided, int i, int* rows, int* tuples, int* colwaves) {
  const int n = strided ? kNumTuneStrided : kNumTuneContig;
  if (i < 0 || i >= n) return fail(SLDG_ERR_ARG, "candidate %d out of range [0, %d)", i, n);
  const int* c = strided ? kTuneStrided[i] : kTuneContig[i];
  if (rows) *rows = c[0];
  if (tuples) *tuples = c[1];
  if (colwaves) *colwaves = c[2];
  return ok();
}

sldg_status sldg_plan_tune(sldg_plan_t p, const sldg_sweep_desc* seq, int nseq,
                           const double* mass0, const void* hi0, double* mass1, void* hi1,
                           int reps, double* best_ms) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (nseq < 0 || (nseq > 0 && !seq) || reps < 1)
    return fail(SLDG_ERR_ARG, "bad sweep sequence or reps (nseq=%d reps=%d)", nseq, reps);
  for (int q = 0; q < nseq; ++q) {
    sldg_status st = check_sweep(p, seq[q].dim, seq[q].shift, seq[q].dep_mask, mass0, hi0, mass1,
                                 hi1);
    if (st != SLDG_OK) return st;
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  if (e != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    return device_error(e, "hipEventCreate");
  }
  const bool timing = p->timing;
  p->timing = false;
  double tuned_ms[kMaxDim];
  bool done[kMaxDim] = {};
  sldg_status st = SLDG_OK;
  for (int q = 0; q < nseq && st == SLDG_OK; ++q) {
    const int dim = seq[q].dim;
    if (done[dim]) {
      if (best_ms) best_ms[q] = tuned_ms[dim];
      continue;
    }
    const bool strided = dim > 0;
    const int n = strided ? kNumTuneStrided : kNumTuneContig;
    // the window form ignores the dimension-0 form choice: its lane variants
    // would time the same launch again
    const bool window = p->n[0] % 4 == 0 &&
                        (((uintptr_t)mass0 | (uintptr_t)hi0 | (uintptr_t)mass1 | (uintptr_t)hi1) &
                         15) == 0;
    const int keep[3] = {p->rows_d[dim], p->tuples_d[dim], p->colwaves_d[dim]};
    // average time of `reps` sweeps in candidate i's shape (after one
    // untimed sweep), or < 0 where the shape does not apply
    auto time_shape = [&](int i, double& avg) -> sldg_status {
      avg = -1.0;
      const int* c = strided ? kTuneStrided[i] : kTuneContig[i];
      p->rows_d[dim] = c[0];
      p->tuples_d[dim] = c[1];
      p->colwaves_d[dim] = c[2];
      if (c[2] & SLDG_SHAPE_STAGED) {   // staged shapes the grid cannot take: not timed
        SweepArgs a{};
        int64_t nt = 0;
        describe(p, dim, seq[q].dep_mask, a, nt);
        if (!staged_fits(p, dim, a, hi0, hi1)) return SLDG_OK;
      }
      sldg_status s1 = run_sweep(p, dim, seq[q].shift, seq[q].dep_mask, mass0, hi0, mass1, hi1);
      if (s1 == SLDG_ERR_UNSUPPORTED) return SLDG_OK;   // shape not launchable on this grid
      if (s1 != SLDG_OK) return s1;
      e = hipEventRecord(e0, p->stream);
      for (int r = 0; r < reps && s1 == SLDG_OK && e == hipSuccess; ++r)
        s1 = run_sweep(p, dim, seq[q].shift, seq[q].dep_mask, mass0, hi0, mass1, hi1);
      if (s1 != SLDG_OK) return s1;
      if (e == hipSuccess) e = hipEventRecord(e1, p->stream);
      if (e == hipSuccess) e = hipEventSynchronize(e1);
      float ms = 0.f;
      if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
      if (e != hipSuccess) return device_error(e, "tuning events");
      avg = ms / reps;
      return SLDG_OK;
    };
    // first pass over every candidate; then the fastest few are timed again,
    // in turn, and ranked by their total, so that one noisy timing does not
    // decide between shapes a few percent apart
    constexpr int kFinal = 3;
    int top[kFinal];
    double topt[kFinal];
    int ntop = 0;
    for (int i = 0; i < n && st == SLDG_OK; ++i) {
      const int* c = strided ? kTuneStrided[i] : kTuneContig[i];
      if (!strided && window && c[0] == 1) continue;
      double avg;
      st = time_shape(i, avg);
      if (st != SLDG_OK || avg < 0) continue;
      int pos = ntop < kFinal ? ntop++ : kFinal;
      if (pos == kFinal) {
        if (avg >= topt[kFinal - 1]) continue;
        pos = kFinal - 1;
      }
      while (pos > 0 && topt[pos - 1] > avg) {
        top[pos] = top[pos - 1];
        topt[pos] = topt[pos - 1];
        --pos;
      }
      top[pos] = i;
      topt[pos] = avg;
    }
    double best = -1.0;
    int bi = -1;
    if (st == SLDG_OK && ntop > 1) {
      double tot[kFinal] = {};
      for (int round = 0; round < 2 && st == SLDG_OK; ++round)
        for (int j = 0; j < ntop && st == SLDG_OK; ++j) {
          double avg;
          st = time_shape(top[j], avg);
          tot[j] += avg;
        }
      for (int j = 0; j < ntop && st == SLDG_OK; ++j)
        if (bi < 0 || tot[j] < 2.0 * best) {
          best = tot[j] / 2.0;
          bi = top[j];
        }
    } else if (st == SLDG_OK && ntop == 1) {
      best = topt[0];
      bi = top[0];
    }
    if (st == SLDG_OK && bi < 0)
      st = fail(SLDG_ERR_UNSUPPORTED, "no launch shape fits the sweep along dim %d", dim);
    if (st != SLDG_OK) {
      p->rows_d[dim] = keep[0];
      p->tuples_d[dim] = keep[1];
      p->colwaves_d[dim] = keep[2];
      break;
    }
    const int* c = strided ? kTuneStrided[bi] : kTuneContig[bi];
    p->rows_d[dim] = c[0];
    p->tuples_d[dim] = c[1];
    p->colwaves_d[dim] = c[2];
    tuned_ms[dim] = best;
    done[dim] = true;
    if (best_ms) best_ms[q] = best;
  }
  p->timing = timing;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return st == SLDG_OK ? ok() : st;
}

int64_t sldg_scale_bytes(sldg_plan_t p) { return p ? 8 * p->n_hi : -1; }

sldg_status sldg_set_scale_headroom(sldg_plan_t p, int binades) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (binades < 0 || binades > 14) return fail(SLDG_ERR_ARG, "headroom %d not in [0, 14]", binades);
  p->scale_headroom = binades;
  return ok();
}

sldg_status sldg_scaled_import(sldg_plan_t p, const double* hi64, void* hi, void* scale) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (p->tier != SLDG_TIER_FP16)
    return fail(SLDG_ERR_UNSUPPORTED, "scaled storage needs an FP16-tier plan");
  if (p->n_hi == 0) return ok();
  if (!hi64 || !hi || !scale) return fail(SLDG_ERR_ARG, "null pointer");
  if ((uintptr_t)scale & 3) return fail(SLDG_ERR_ARG, "scale block must be 4-byte aligned");
  const int64_t b64 = p->n_hi * p->cells * 8, sb = 8 * p->n_hi;
  if (overlap(hi64, b64, hi, p->hi_bytes) || overlap(hi64, b64, scale, sb) ||
      overlap(hi, p->hi_bytes, scale, sb))
    return fail(SLDG_ERR_ALIAS, "import buffers overlap");
  if (p->n_hi > 65535) return fail(SLDG_ERR_UNSUPPORTED, "too many planes for the import grid");
  sldg_status st = ensure_part(p, p->n_hi * (int64_t)kImportSlots);
  if (st != SLDG_OK) return st;
  ScaleBlock sc = scale_view(p, scale);
  hipError_t e = launch_scale_import(hi64, p->n_hi, p->cells, p->scale_headroom, p->d_part,
                                     kImportSlots, hi, sc.exp, sc.amax, p->stream);
  if (e != hipSuccess) return device_error(e, "scaled import launch");
  return ok();
}

sldg_status sldg_scaled_export(sldg_plan_t p, const void* hi, const void* scale, double* hi64) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (p->tier != SLDG_TIER_FP16)
    return fail(SLDG_ERR_UNSUPPORTED, "scaled storage needs an FP16-tier plan");
  if (p->n_hi == 0) return ok();
  if (!hi64 || !hi || !scale) return fail(SLDG_ERR_ARG, "null pointer");
  const int64_t b64 = p->n_hi * p->cells * 8;
  if (overlap(hi64, b64, hi, p->hi_bytes) || overlap(hi64, b64, scale, 8 * p->n_hi))
    return fail(SLDG_ERR_ALIAS, "export buffers overlap");
  ScaleBlock sc = scale_view(p, scale);
  hipError_t e = launch_scale_export(hi, p->n_hi, p->cells, sc.exp, hi64, p->stream);
  if (e != hipSuccess) return device_error(e, "scaled export launch");
  return ok();
}

sldg_status sldg_advect_dim_scaled(sldg_plan_t p, int dim, const double* shift,
                                   uint32_t dep_mask, const double* in_mass, const void* in_hi,
                                   const void* in_scale, double* out_mass, void* out_hi,
                                   void* out_scale) {
  sldg_status st = check_sweep(p, dim, shift, dep_mask, in_mass, in_hi, out_mass, out_hi);
  if (st != SLDG_OK) return st;
  const void* bufs[4] = {in_mass, in_hi, out_mass, out_hi};
  const int64_t sizes[4] = {p->lo_bytes, p->hi_bytes, p->lo_bytes, p->hi_bytes};
  st = check_scaled(p, in_scale, out_scale, bufs, sizes, 4);
  if (st != SLDG_OK) return st;
  st = run_sweep(p, dim, shift, dep_mask, in_mass, in_hi, out_mass, out_hi, false, in_scale,
                 out_scale);
  return st == SLDG_OK ? ok() : st;
}

sldg_status sldg_split_steps_scaled(sldg_plan_t p, const sldg_sweep_desc* seq, int nseq,
                                    int nsteps, double* mass0, void* hi0, void* scale0,
                                    double* mass1, void* hi1, void* scale1,
                                    int* result_buffer) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (nseq < 0 || nsteps < 0 || (nseq > 0 && !seq))
    return fail(SLDG_ERR_ARG, "bad sweep sequence (nseq=%d nsteps=%d)", nseq, nsteps);
  double* m[2] = {mass0, mass1};
  void* h[2] = {hi0, hi1};
  void* sc[2] = {scale0, scale1};
  const void* bufs[4] = {mass0, hi0, mass1, hi1};
  const int64_t sizes[4] = {p->lo_bytes, p->hi_bytes, p->lo_bytes, p->hi_bytes};
  sldg_status st = check_scaled(p, scale0, scale1, bufs, sizes, 4);
  if (st != SLDG_OK) return st;
  for (int q = 0; q < nseq; ++q)
    for (int b = 0; b < 2; ++b) {
      st = check_sweep(p, seq[q].dim, seq[q].shift, seq[q].dep_mask, m[b], h[b], m[1 - b],
                       h[1 - b]);
      if (st != SLDG_OK) return st;
    }
  int cur = 0;
  for (int n = 0; n < nsteps; ++n)
    for (int q = 0; q < nseq; ++q) {
      st = run_sweep(p, seq[q].dim, seq[q].shift, seq[q].dep_mask, m[cur], h[cur], m[1 - cur],
                     h[1 - cur], false, sc[cur], sc[1 - cur]);
      if (st != SLDG_OK) return st;
      cur = 1 - cur;
    }
  if (result_buffer) *result_buffer = cur;
  return ok();
}

sldg_status sldg_device_copy(const void* src, void* dst, int64_t bytes, void* stream) {
  if (!src || !dst) return fail(SLDG_ERR_ARG, "null pointer");
  if (bytes < 0 || (bytes & 15) || (((uintptr_t)src | (uintptr_t)dst) & 15))
    return fail(SLDG_ERR_ARG, "copy needs a multiple of 16 bytes and 16-byte aligned pointers");
  if (overlap(src, bytes, dst, bytes)) return fail(SLDG_ERR_ALIAS, "copy buffers overlap");
  hipError_t e = launch_copy16(src, dst, bytes / 16, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return device_error(e, "copy launch");
  return ok();
}

namespace {

// Gauss-Legendre nodes (ascending) and weights of the o-point rule, o = 2..4,
// from their closed forms.
void gauss_rule(int o, double* x, double* w) {
  if (o == 2) {
    const double a = 1.0 / std::sqrt(3.0);
    x[0] = -a; x[1] = a;
    w[0] = w[1] = 1.0;
  } else if (o == 3) {
    const double a = std::sqrt(0.6);
    x[0] = -a; x[1] = 0.0; x[2] = a;
    w[0] = w[2] = 5.0 / 9.0;
    w[1] = 8.0 / 9.0;
  } else {
    const double r = 2.0 / 7.0 * std::sqrt(6.0 / 5.0);
    const double outer = std::sqrt(3.0 / 7.0 + r), inner = std::sqrt(3.0 / 7.0 - r);
    const double wo = (18.0 - std::sqrt(30.0)) / 36.0, wi = (18.0 + std::sqrt(30.0)) / 36.0;
    x[0] = -outer; x[1] = -inner; x[2] = inner; x[3] = outer;
    w[0] = w[3] = wo;
    w[1] = w[2] = wi;
  }
}

}  // namespace

sldg_status sldg_advect_dim_collocated(sldg_plan_t p, int dim, int tdim, const double* node_shift,
                                       const double* in_mass, const void* in_hi,
                                       double* out_mass, void* out_hi) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (tdim < 0 || tdim >= p->ndim || tdim == dim)
    return fail(SLDG_ERR_ARG, "transverse dim %d invalid for the sweep along %d", tdim, dim);
  sldg_status st = check_sweep(p, dim, node_shift, 1u << tdim, in_mass, in_hi, out_mass, out_hi);
  if (st != SLDG_OK) return st;
  const int o = p->o;
  const int64_t nent = p->n[tdim] * o;
  if ((p->lo_bytes > 0 && overlap(node_shift, 8 * nent, out_mass, p->lo_bytes)) ||
      (p->hi_bytes > 0 && overlap(node_shift, 8 * nent, out_hi, p->hi_bytes)))
    return fail(SLDG_ERR_ALIAS, "node_shift overlaps an output buffer");
  if (nent > p->table_cap) return fail(SLDG_ERR_ARG, "too many node entries for the plan tables");
  hipError_t e = launch_line_tables(p->k, nent, p->n[dim], node_shift, p->d_s, p->d_ab, true,
                                    false, p->stream);
  if (e != hipSuccess) return device_error(e, "line-table launch");
  ColArgs a{};
  a.in_lo = in_mass;
  a.in_hi = in_hi;
  a.out_lo = out_mass;
  a.out_hi = out_hi;
  a.pmap = p->d_pmap;
  a.s_tab = p->d_s;
  a.ab_tab = p->d_ab;
  a.ab_cs = nent;
  a.cells = p->cells;
  a.ndim = p->ndim;
  a.d = dim;
  a.t = tdim;
  int64_t Pd = 1, Pt = 1;
  int32_t msd = 1, mst = 1;
  for (int f = 0; f < dim; ++f) { Pd *= p->n[f]; msd *= o; }
  for (int f = 0; f < tdim; ++f) { Pt *= p->n[f]; mst *= o; }
  a.Pd = Pd;
  a.Nd = p->n[dim];
  a.Pt = Pt;
  a.Nt = p->n[tdim];
  a.fPd = FastDiv::make((uint32_t)Pd);
  a.fNd = FastDiv::make((uint32_t)a.Nd);
  a.fPt = FastDiv::make((uint32_t)Pt);
  a.fNt = FastDiv::make((uint32_t)a.Nt);
  a.n_lo = (int32_t)p->n_lo;
  a.wide = p->ndouble > 1 ? 1 : 0;
  a.msd = msd;
  a.mst = mst;
  int32_t groups = 1;
  for (int f = 0; f < p->ndim - 2; ++f) groups *= o;
  a.ngroups = groups;
  double x[4], w[4];
  gauss_rule(o, x, w);
  for (int q = 0; q < o; ++q) {
    double pm = 1.0, pc = x[q];          // P_0, P_1 (Bonnet's recurrence)
    for (int j = 0; j < o; ++j) {
      double pj;
      if (j == 0) pj = 1.0;
      else if (j == 1) pj = x[q];
      else {
        const double pn = ((2 * (j - 1) + 1) * x[q] * pc - (j - 1) * pm) / j;
        pm = pc;
        pc = pn;
        pj = pn;
      }
      a.P[j][q] = pj;
      a.back[j][q] = 0.5 * (2 * j + 1) * w[q] * pj;
    }
  }
  e = launch_colloc(p->k, (int)p->tier, a, p->stream);
  if (e == hipErrorInvalidConfiguration)
    return fail(SLDG_ERR_UNSUPPORTED, "collocated sweep: grid too large for one launch");
  if (e != hipSuccess) return device_error(e, "collocated sweep launch");
  return ok();
}

// Grows the plan's field scratch to `need` doubles (freeing the old one waits
// for the device, so earlier solves that used the old buffer have finished).
static sldg_status ensure_field(sldg_plan_t p, int64_t need) {
  if (need <= p->field_cap) return SLDG_OK;
  if (p->d_field) dev_free(p->d_field);
  p->d_field = nullptr;
  p->field_cap = 0;
  hipError_t e = dev_malloc(&p->d_field, sizeof(double) * (size_t)need);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(SLDG_ERR_NOMEM, "field scratch: %s", hipGetErrorString(e));
  }
  p->field_cap = need;
  return SLDG_OK;
}

// Arguments of a 1D-1V field solve: checks them and fills the mode planes.
static sldg_status poisson_shift_args(sldg_plan_t p, const double* mass, const void* hi,
                                      double hx, double hv, double dt, double* shift_out,
                                      double* field_out, FieldPlanes& fp) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (p->ndim != 2) return fail(SLDG_ERR_ARG, "the field solve needs an (x, v) plan (ndim = 2)");
  if (!(hx > 0.0) || !(hv > 0.0) || !std::isfinite(dt))
    return fail(SLDG_ERR_ARG, "hx, hv must be > 0 and dt finite");
  if (!shift_out) return fail(SLDG_ERR_ARG, "null shift_out");
  if (p->n_lo > 0 && !mass) return fail(SLDG_ERR_ARG, "null mass");
  if (p->n_hi > 0 && !hi) return fail(SLDG_ERR_ARG, "null hi");
  const int64_t ob = 8 * p->n[0];
  const void* outs[2] = {shift_out, field_out};
  for (int i = 0; i < 2; ++i) {
    if (!outs[i]) continue;
    if ((p->lo_bytes > 0 && overlap(outs[i], ob, mass, p->lo_bytes)) ||
        (p->hi_bytes > 0 && overlap(outs[i], ob, hi, p->hi_bytes)))
      return fail(SLDG_ERR_ALIAS, "field output overlaps the state");
  }
  if (field_out && overlap(shift_out, ob, field_out, ob))
    return fail(SLDG_ERR_ALIAS, "shift_out overlaps field_out");
  // planes of the modes (j, 0): mode id j
  fp = FieldPlanes{};
  for (int j = 0; j < p->o; ++j) {
    const int32_t v = p->h_pmap[j];
    fp.lo[j] = v < 0 ? 1 : 0;
    fp.plane[j] = v < 0 ? static_cast<const void*>(mass + (int64_t)(-1 - v) * p->cells)
                        : static_cast<const void*>(static_cast<const char*>(hi) +
                                                   (int64_t)v * p->cells * elem_size(p->tier));
  }
  return SLDG_OK;
}

sldg_status sldg_poisson_shift(sldg_plan_t p, const double* mass, const void* hi, double hx,
                               double hv, double dt, double* shift_out, double* field_out) {
  FieldPlanes fp;
  sldg_status st = poisson_shift_args(p, mass, hi, hx, hv, dt, shift_out, field_out, fp);
  if (st != SLDG_OK) return st;
  const int32_t nx = (int32_t)p->n[0], nv = (int32_t)p->n[1];
  st = ensure_field(p, field_scratch_doubles(p->o, nx, nv));
  if (st != SLDG_OK) return st;
  hipError_t e = launch_field((int)p->tier, fp, p->o, nx, nv, hx, hv, dt, p->d_field, shift_out,
                              field_out, p->stream);
  if (e != hipSuccess) return device_error(e, "field launch");
  return ok();
}

sldg_status sldg_poisson_shift_noalloc(sldg_plan_t p, const double* mass, const void* hi,
                                       double hx, double hv, double dt, double* shift_out,
                                       double* field_out) {
  FieldPlanes fp;
  sldg_status st = poisson_shift_args(p, mass, hi, hx, hv, dt, shift_out, field_out, fp);
  if (st != SLDG_OK) return st;
  const int32_t nx = (int32_t)p->n[0], nv = (int32_t)p->n[1];
  const int64_t need = field_scratch_doubles(p->o, nx, nv);
  if (need > kStaticFieldDoubles)
    return fail(SLDG_ERR_UNSUPPORTED,
                "allocation-free field solve: N_x = %d at degree %d needs %lld doubles of "
                "scratch, more than the static %lld (use sldg_poisson_shift)",
                (int)nx, p->k, (long long)need, (long long)kStaticFieldDoubles);
  double* buf = (p->device >= 0 && p->device < kMaxDevices) ? g_scratch_ptr[p->device] : nullptr;
  if (!buf)
    return fail(SLDG_ERR_UNSUPPORTED, "allocation-free field solve: no static scratch on device %d",
                p->device);
  hipError_t e = launch_field((int)p->tier, fp, p->o, nx, nv, hx, hv, dt, buf, shift_out,
                              field_out, p->stream);
  if (e != hipSuccess) return device_error(e, "field launch");
  return ok();
}

sldg_status sldg_vlasov_poisson_steps(sldg_plan_t p, int nsteps, const double* shift_x, double hx,
                                      double hv, double dt, double* shift_v, double* mass0,
                                      void* hi0, double* mass1, void* hi1, int* result_buffer) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (p->ndim != 2) return fail(SLDG_ERR_ARG, "Vlasov-Poisson steps need an (x, v) plan");
  if (nsteps < 0) return fail(SLDG_ERR_ARG, "nsteps %d < 0", nsteps);
  if (!shift_x || !shift_v) return fail(SLDG_ERR_ARG, "null shift pointer");
  double* m[2] = {mass0, mass1};
  void* h[2] = {hi0, hi1};
  for (int b = 0; b < 2; ++b) {
    sldg_status st = check_sweep(p, 0, shift_x, 2u, m[b], h[b], m[1 - b], h[1 - b]);
    if (st == SLDG_OK) st = check_sweep(p, 1, shift_v, 1u, m[b], h[b], m[1 - b], h[1 - b]);
    if (st != SLDG_OK) return st;
  }
  const int64_t ob = 8 * p->n[0];
  for (int b = 0; b < 2; ++b)
    if ((p->lo_bytes > 0 && overlap(shift_v, ob, m[b], p->lo_bytes)) ||
        (p->hi_bytes > 0 && overlap(shift_v, ob, h[b], p->hi_bytes)))
      return fail(SLDG_ERR_ALIAS, "shift_v overlaps a state buffer");
  int cur = 0;
  StrangArgs xs{};
  int64_t nblocks = 0;
  const int64_t N0 = p->n[0], N1 = p->n[1];
  const int64_t second = N1;       // tables: the X table by entries, then the one in use
  if (nsteps > 1 && strang_eligible(p, xs, nblocks) && N1 + std::max(N0, N1) <= p->table_cap &&
      !overlap(shift_x, 8 * N1, shift_v, ob)) {
    // The end of a step and the start of the next, V X X, are one pass; the
    // first X and the last V and X run alone, so that the result lands in the
    // buffer that three sweeps a step leave it in.  The X displacements are
    // fixed over the call (unless a field solve writes over them): their table
    // is computed once.
    const int64_t E = 2LL * p->o * p->o;
    auto table = [&](int dim, const double* shift, bool by_entry) -> sldg_status {
      const int64_t at = by_entry ? 0 : second;
      const hipError_t e = launch_line_tables(p->k, dim ? N0 : N1, p->n[dim], shift, p->d_s + at,
                                              p->d_ab + E * at, !by_entry, false, p->stream);
      return e == hipSuccess ? SLDG_OK : device_error(e, "line-table launch");
    };
    auto sweep = [&](int dim, const double* shift, uint32_t mask) -> sldg_status {
      sldg_status st = table(dim, shift, false);
      if (st == SLDG_OK)
        st = run_sweep(p, dim, shift, mask, m[cur], h[cur], m[1 - cur], h[1 - cur], false, nullptr,
                       nullptr, second);
      if (st == SLDG_OK) cur = 1 - cur;
      return st;
    };
    const uint32_t mask[3] = {0, 1u, 2u};
    const int64_t at[3] = {0, second, 0};
    sldg_status st = table(0, shift_x, true);
    if (st == SLDG_OK) st = sweep(0, shift_x, 2u);
    for (int n = 0; n < nsteps && st == SLDG_OK; ++n) {
      st = sldg_poisson_shift(p, m[cur], h[cur], hx, hv, dt, shift_v, nullptr);
      if (st != SLDG_OK) break;
      if (n + 1 < nsteps) {
        st = table(1, shift_v, false);
        if (st == SLDG_OK)
          st = run_strang(p, 2, mask, at, m[cur], h[cur], m[1 - cur], h[1 - cur]);
        cur = 1 - cur;
      } else {
        st = sweep(1, shift_v, 1u);
        if (st == SLDG_OK) st = sweep(0, shift_x, 2u);
      }
    }
    if (st != SLDG_OK) return st;
    if (result_buffer) *result_buffer = cur;
    return ok();
  }
  for (int n = 0; n < nsteps; ++n) {
    // X(dt/2), field from the state, V(dt), X(dt/2)
    sldg_status st = run_sweep(p, 0, shift_x, 2u, m[cur], h[cur], m[1 - cur], h[1 - cur]);
    if (st != SLDG_OK) return st;
    cur = 1 - cur;
    st = sldg_poisson_shift(p, m[cur], h[cur], hx, hv, dt, shift_v, nullptr);
    if (st != SLDG_OK) return st;
    st = run_sweep(p, 1, shift_v, 1u, m[cur], h[cur], m[1 - cur], h[1 - cur]);
    if (st != SLDG_OK) return st;
    cur = 1 - cur;
    st = run_sweep(p, 0, shift_x, 2u, m[cur], h[cur], m[1 - cur], h[1 - cur]);
    if (st != SLDG_OK) return st;
    cur = 1 - cur;
  }
  if (result_buffer) *result_buffer = cur;
  return ok();
}

sldg_status sldg_poisson_shift_2d(sldg_plan_t p, const double* mass, const void* hi,
                                  const double* h, double dt, double* shift_v1, double* shift_v2,
                                  double* field_out) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (p->ndim != 4)
    return fail(SLDG_ERR_ARG, "the 2D field solve needs an (x1, x2, v1, v2) plan (ndim = 4)");
  if (!h) return fail(SLDG_ERR_ARG, "null cell widths");
  for (int d = 0; d < 4; ++d)
    if (!(h[d] > 0.0) || !std::isfinite(h[d]))
      return fail(SLDG_ERR_ARG, "cell width h[%d] = %g must be finite and > 0", d, h[d]);
  if (!std::isfinite(dt)) return fail(SLDG_ERR_ARG, "dt must be finite");
  if (!shift_v1 || !shift_v2) return fail(SLDG_ERR_ARG, "null shift output");
  if (p->n[0] > kMaxDft || p->n[1] > kMaxDft)
    return fail(SLDG_ERR_UNSUPPORTED, "2D field solve: N1, N2 must be <= %d", (int)kMaxDft);
  const int32_t v = p->h_pmap[0];
  if (v < 0 ? !mass : !hi) return fail(SLDG_ERR_ARG, "null state pointer");
  const int64_t nxx = p->n[0] * p->n[1];
  const int64_t ob = 8 * nxx;
  const void* outs[3] = {shift_v1, shift_v2, field_out};
  const int64_t len[3] = {ob, ob, 2 * ob};
  for (int i = 0; i < 3; ++i) {
    if (!outs[i]) continue;
    if ((p->lo_bytes > 0 && overlap(outs[i], len[i], mass, p->lo_bytes)) ||
        (p->hi_bytes > 0 && overlap(outs[i], len[i], hi, p->hi_bytes)))
      return fail(SLDG_ERR_ALIAS, "field output overlaps the state");
    for (int j = 0; j < i; ++j)
      if (outs[j] && overlap(outs[i], len[i], outs[j], len[j]))
        return fail(SLDG_ERR_ALIAS, "field outputs overlap each other");
  }
  Field2Args a{};
  a.lo0 = v < 0 ? 1 : 0;
  a.plane0 = v < 0 ? static_cast<const void*>(mass + (int64_t)(-1 - v) * p->cells)
                   : static_cast<const void*>(static_cast<const char*>(hi) +
                                              (int64_t)v * p->cells * elem_size(p->tier));
  a.n1 = (int32_t)p->n[0];
  a.n2 = (int32_t)p->n[1];
  a.nslab = p->n[2] * p->n[3];
  a.h1 = h[0];
  a.h2 = h[1];
  a.hv1 = h[2];
  a.hv2 = h[3];
  a.dt = dt;
  a.shift1 = shift_v1;
  a.shift2 = shift_v2;
  a.field = field_out;
  sldg_status st = ensure_field(p, field2_scratch_doubles(a.n1, a.n2, a.nslab));
  if (st != SLDG_OK) return st;
  hipError_t e = launch_field2((int)p->tier, a, p->d_field, p->stream);
  if (e != hipSuccess) return device_error(e, "2D field launch");
  return ok();
}

sldg_status sldg_vlasov_poisson_steps_2d2v(sldg_plan_t p, int nsteps, const double* shift_x1,
                                           const double* shift_x2, const double* h, double dt,
                                           double* shift_v1, double* shift_v2, double* mass0,
                                           void* hi0, double* mass1, void* hi1,
                                           int* result_buffer) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (p->ndim != 4) return fail(SLDG_ERR_ARG, "2D-2V Vlasov-Poisson steps need ndim = 4");
  if (nsteps < 0) return fail(SLDG_ERR_ARG, "nsteps %d < 0", nsteps);
  if (!shift_x1 || !shift_x2 || !shift_v1 || !shift_v2)
    return fail(SLDG_ERR_ARG, "null shift pointer");
  double* m[2] = {mass0, mass1};
  void* hh[2] = {hi0, hi1};
  // x1 moves with v1 (dep dim 2), x2 with v2 (dep dim 3); v1, v2 with E(x1, x2)
  const unsigned dep[4] = {1u << 2, 1u << 3, 3u, 3u};
  const double* sh[4] = {shift_x1, shift_x2, shift_v1, shift_v2};
  for (int b = 0; b < 2; ++b)
    for (int d = 0; d < 4; ++d) {
      sldg_status st = check_sweep(p, d, sh[d], dep[d], m[b], hh[b], m[1 - b], hh[1 - b]);
      if (st != SLDG_OK) return st;
    }
  const int64_t ob = 8 * p->n[0] * p->n[1];
  for (int b = 0; b < 2; ++b)
    for (double* s : {shift_v1, shift_v2})
      if ((p->lo_bytes > 0 && overlap(s, ob, m[b], p->lo_bytes)) ||
          (p->hi_bytes > 0 && overlap(s, ob, hh[b], p->hi_bytes)))
        return fail(SLDG_ERR_ALIAS, "a v shift table overlaps a state buffer");
  if (overlap(shift_v1, ob, shift_v2, ob)) return fail(SLDG_ERR_ALIAS, "shift_v1 overlaps shift_v2");
  int cur = 0;
  // The x displacements are fixed over the call: their tables are computed
  // once, before the steps, and those of the two v sweeps in one launch after
  // each field solve, where all four fit the plan's table storage together.
  const int64_t o2 = (int64_t)p->o * p->o;
  const int64_t nx = p->n[2] + p->n[3], nv = p->n[0] * p->n[1];
  bool tables = nx + 2 * nv <= p->table_cap;
  for (const double* v : {shift_v1, shift_v2})    // (unless a field solve writes over them)
    if (overlap(shift_x1, 8 * p->n[2], v, ob) || overlap(shift_x2, 8 * p->n[3], v, ob))
      tables = false;
  int64_t pre[4] = {-1, -1, -1, -1};
  ColPairArgs cp{};
  int64_t nblocks = 0;
  const bool vpair = tables && nx + 2 * nv + kPairFlags <= p->table_cap &&
                     colpair_eligible(p, 2, dep[2], dep[3], cp, nblocks);
  auto compute = [&](int d0, int64_t at) -> sldg_status {
    TableSet set{};
    set.count = 2;
    for (int i = 0; i < 2; ++i) {
      const int64_t n = d0 == 0 ? p->n[2 + i] : nv;
      set.first[i + 1] = set.first[i] + n;
      set.period[i] = p->n[d0 + i];
      set.sigma[i] = sh[d0 + i];
      pre[d0 + i] = at + set.first[i];
    }
    if (d0 == 2 && vpair) set.pair = pair_decision(p, 2, sh[2], dep[2], sh[3], dep[3], 0);
    const hipError_t e =
        launch_line_tables_set(p->k, set, p->d_s + at, p->d_ab + 2 * o2 * at, p->stream);
    return e == hipSuccess ? SLDG_OK : device_error(e, "line-table launch");
  };
  auto sweep = [&](int d) {
    sldg_status st = run_sweep(p, d, sh[d], dep[d], m[cur], hh[cur], m[1 - cur], hh[1 - cur], false,
                               nullptr, nullptr, pre[d]);
    if (st == SLDG_OK) cur = 1 - cur;
    return st;
  };
  // X1 X2 as one fused pass where it can run (two passes a step, as four
  // sweeps, end in the buffer they started from), and V1 V2 (one pass a step: a
  // caller that does not ask for the result's buffer finds it in buffer 0, the
  // last of an odd number of steps running the two sweeps)
  const char* why = nullptr;
  const bool pair =
      p->fuse && xy_eligible(p, dep[0], dep[1], m[0], hh[0], m[1], hh[1], &why);
  auto x_sweeps = [&] {
    sldg_status st;
    if (pair) {
      st = run_xy(p, sh[0], dep[0], sh[1], dep[1], m[cur], hh[cur], m[1 - cur], hh[1 - cur], pre[0],
                  pre[1]);
      if (st == SLDG_OK) cur = 1 - cur;
    } else {
      st = sweep(0);
      if (st == SLDG_OK) st = sweep(1);
    }
    return st;
  };
  auto v_sweeps = [&](bool last) {
    sldg_status st;
    if (vpair && !(last && !result_buffer && nsteps % 2)) {
      st = run_colpair(p, 2, dep[2], dep[3], pre[2], pre[3], 0, m[cur], hh[cur], m[1 - cur],
                       hh[1 - cur]);
      if (st == SLDG_OK) cur = 1 - cur;
    } else {
      st = sweep(2);
      if (st == SLDG_OK) st = sweep(3);
    }
    return st;
  };
  sldg_status st = SLDG_OK;
  if (tables && nsteps > 0 && (st = compute(0, 0)) != SLDG_OK) return st;
  for (int n = 0; n < nsteps; ++n) {
    // X1(dt/2) X2(dt/2), the field of the state, V1(dt) V2(dt), X1(dt/2) X2(dt/2)
    if ((st = x_sweeps()) != SLDG_OK) return st;
    st = sldg_poisson_shift_2d(p, m[cur], hh[cur], h, dt, shift_v1, shift_v2, nullptr);
    if (st == SLDG_OK && tables) st = compute(2, nx);
    if (st != SLDG_OK) return st;
    if ((st = v_sweeps(n + 1 == nsteps)) != SLDG_OK) return st;
    if ((st = x_sweeps()) != SLDG_OK) return st;
  }
  if (result_buffer) *result_buffer = cur;
  return ok();
}

sldg_status sldg_device_plane_copy(const void* src, void* dst, int64_t plane_bytes, int nplanes,
                                   int planes_per_thread, void* stream) {
  if (!src || !dst) return fail(SLDG_ERR_ARG, "null pointer");
  if (plane_bytes < 0 || (plane_bytes & 15) || nplanes < 0 || planes_per_thread < 1 ||
      (((uintptr_t)src | (uintptr_t)dst) & 15))
    return fail(SLDG_ERR_ARG, "plane copy needs 16-byte multiples and alignment, T >= 1");
  const int64_t bytes = plane_bytes * nplanes;
  if (overlap(src, bytes, dst, bytes)) return fail(SLDG_ERR_ALIAS, "copy buffers overlap");
  hipError_t e = launch_plane_copy16(src, dst, plane_bytes / 16, nplanes, planes_per_thread,
                                     static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return device_error(e, "plane copy launch");
  return ok();
}

sldg_status sldg_mass_device(sldg_plan_t p, const double* mass, double* out_dev) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (p->n_lo < 1) return fail(SLDG_ERR_ARG, "mode 0 is not stored in FP64 (ndouble = 0)");
  if (!mass || !out_dev) return fail(SLDG_ERR_ARG, "null pointer");
  if (overlap(out_dev, 16, mass, p->cells * 8))
    return fail(SLDG_ERR_ALIAS, "out_dev overlaps the mass array");
  hipError_t e = launch_mass(mass, p->cells, p->d_mass_part, p->mass_nblocks, out_dev, p->stream);
  if (e != hipSuccess) return device_error(e, "mass launch");
  return ok();
}

sldg_status sldg_mass(sldg_plan_t p, const double* mass, double out[2]) {
  if (!p) return fail(SLDG_ERR_ARG, "plan is NULL");
  if (p->n_lo < 1) return fail(SLDG_ERR_ARG, "mode 0 is not stored in FP64 (ndouble = 0)");
  if (!mass || !out) return fail(SLDG_ERR_ARG, "null pointer");
  hipError_t e = launch_mass(mass, p->cells, p->d_mass_part, p->mass_nblocks, p->d_mass_out,
                             p->stream);
  if (e != hipSuccess) return device_error(e, "mass launch");
  e = hipMemcpyAsync(p->h_mass_out, p->d_mass_out, sizeof(double) * 2, hipMemcpyDeviceToHost,
                     p->stream);
  if (e != hipSuccess) return device_error(e, "mass copy");
  e = hipStreamSynchronize(p->stream);
  if (e != hipSuccess) return device_error(e, "mass synchronize");
  out[0] = p->h_mass_out[0];
  out[1] = p->h_mass_out[1];
  return ok();
}

}  // extern "C"
