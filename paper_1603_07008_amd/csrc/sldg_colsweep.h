// One projection sweep along a dimension d >= 1 with whole lines in LDS (L.
// Einkemmer, arXiv 1603.07008, section II-A update rule), run where a device
// flag says so: the two sweeps of a column pair (sldg_colpair.h) whose
// displacements are too spread for the fused pass.
//
// A workgroup takes C neighbouring columns (cells below d) of one slab and one
// spectator tuple, loads their whole lines (N rows of the o modes) row by row,
// and computes every output cell from LDS, where the rows of a lane's own shift
// cost no more than equal ones.  All of a tile's sources are read before its
// first output is stored, so a sweep may run in place: the pair's second sweep
// does, and ends in the buffer that the fused pass would have written.  The
// update is computed as the other kernels do, to the same bits.
//
// Bound by memory: each value is read and written once, in runs of C cells.  Both
// sweeps of 48^4 cells, k = 2, FP32 1.54 ms, BF16 0.89, FP64 2.78, at any
// displacements; the plan's sweeps 1.40, 0.74 and 2.65 ms where the pair's columns
// span 4 cells, 1.77, 0.99 and 3.44 ms at 14, and the fused pass 4.98, 2.80 and
// 6.07 ms there.  24^4, k = 3, FP32 0.36 (0.44 at 15 cells); tiles of 64 instead of
// 128 columns took BF16 0.97.  Loads of 16 bytes a lane, one plane after the
// other, were slower (48^4, k = 2, BF16 1.09).  Persistent workgroups, so that a
// launch whose flag is clear costs a launch; XCD runs of 16 tiles gain 6% on uneven
// rows (30 x 30 x 50 x 20).
#pragma once

#include "sldg_strang.h"

namespace sldg {

struct ColSweepArgs {
  const double* in_lo;       // FP64 plane of mode 0 (n_lo == 1), or unused
  const void* in_hi;         // the other modes, storage type of the tier
  double* out_lo;            // may be the inputs
  void* out_hi;
  int32_t n_lo;
  int64_t cells;             // cells of the grid (plane length)
  int32_t P, N, Q;           // cells below d, extent of d, cells above
  int32_t ms;                // o^d: mode-id stride of j_d
  int32_t logc, logc64;      // columns per tile, and at a time of a tuple with the FP64
                             // mode (log2)
  int32_t ntile;             // column tiles of a slab
  int32_t items;             // tiles x slabs x spectator tuples
  float one;                 // 1.0f: the FP16 tier's unit scale
  FastDiv ftile, fQ;
  const int32_t* s;          // line table, component-major
  const double* ab;
  int64_t cs;
  LineMap map;
  const int32_t* flag;       // the sweep runs where *flag != 0
};

constexpr int64_t kColSweepLds = 80 * 1024;       // two workgroups a CU at least
constexpr int64_t kColSweepLdsMax = 160 * 1024;   // ... where 8 columns take more

// Columns per tile (256 bytes of a row, where there are as many columns) and their
// LDS bytes, for a's P and N; false: lines too long.  The one tuple with an FP64
// mode takes fewer columns at a time, so that it sets no tile's size.
inline bool colsweep_tiles(ColSweepArgs& a, int o, int64_t elem, int64_t& lds) {
  for (a.logc = elem == 2 && a.P >= 256 ? 7 : 6; a.logc >= 3; --a.logc) {
    lds = ((int64_t)a.N * o * elem) << a.logc;
    if (lds > (a.logc == 3 ? kColSweepLdsMax : kColSweepLds)) continue;
    a.logc64 = a.logc;
    while (a.logc64 > 0 && ((int64_t)a.N * (8 + (o - 1) * elem)) << a.logc64 > lds) --a.logc64;
    return ((int64_t)a.N * (8 + (o - 1) * elem)) << a.logc64 <= lds;
  }
  return false;
}

template <int K, int TIER, int H64>
__device__ __forceinline__ void colsweep_tile(const ColSweepArgs& a, int32_t first, int32_t logc,
                                              int32_t slab, int32_t spec, unsigned char* smem) {
  constexpr int O = K + 1;
  using T = typename Tier<TIER>::T;
  const int32_t N = a.N, C = 1 << logc, P = a.P;
  const int32_t c = (int32_t)threadIdx.x & (C - 1), r0 = (int32_t)threadIdx.x >> logc;
  const int32_t step = 256 >> logc;
  const int32_t col = first + c;
  const bool act = col < P;
  double* d64 = reinterpret_cast<double*>(smem);             // [N][C]
  T* buf = reinterpret_cast<T*>(smem + (H64 ? 8LL * N * C : 0));   // [O - H64][N][C]
  const int32_t low = spec % a.ms, m0 = low + (spec - low) * O;
  const int64_t base = (int64_t)slab * N * P + col;
  auto plane = [&](int l) {
    return as_global(reinterpret_cast<const T*>(a.in_hi)) +
           ((int64_t)m0 + (int64_t)l * a.ms - a.n_lo) * a.cells + base;
  };
  if (act) {
#pragma unroll 4
    for (int32_t r = r0; r < N; r += step) {
      const int64_t at = (int64_t)r * P;
      if (H64) d64[r * C + c] = as_global(a.in_lo)[base + at];
#pragma unroll
      for (int l = H64; l < O; ++l) buf[((l - H64) * N + r) * C + c] = plane(l)[at];
    }
  }
  __syncthreads();
  if (act) {
    const int32_t t = table_index(a.map, col, slab);
    const int32_t s = as_global(a.s)[t];
    Mat<K, TIER> M;
    Rows64<K, 1> R;
    const auto* ab = as_global(a.ab) + t;
#pragma unroll
    for (int j = 0; j < O; ++j)
#pragma unroll
      for (int l = 0; l < O; ++l) {
        const double A = ab[(j * O + l) * a.cs], B = ab[(O * O + j * O + l) * a.cs];
        M.Aa[j][l] = (typename Tier<TIER>::Acc)A;
        M.Ba[j][l] = (typename Tier<TIER>::Acc)B;
        if (H64 && j == 0) {
          R.A[0][l] = A;
          R.B[0][l] = B;
        }
      }
    T* const out = reinterpret_cast<T*>(a.out_hi);
    for (int32_t r = r0; r < N; r += step) {
      int32_t x = r - s;
      x = x < 0 ? x + N : x;
      const int32_t y = x == 0 ? N - 1 : x - 1;
      Raw<K, TIER, H64> xs, ys;
#pragma unroll
      for (int l = 0; l < O; ++l) {
        raw_set<K, TIER, H64>(xs, l, l < H64 ? T(0) : buf[((l - H64) * N + x) * C + c],
                              l < H64 ? d64[x * C + c] : 0.0, a.one);
        raw_set<K, TIER, H64>(ys, l, l < H64 ? T(0) : buf[((l - H64) * N + y) * C + c],
                              l < H64 ? d64[y * C + c] : 0.0, a.one);
      }
      T w[O];
      double w64 = 0.0;
      strang_tuple<K, TIER, H64>(M, R, xs, ys, w, w64, a.one);
      const int64_t at = base + (int64_t)r * P;
      if (H64) a.out_lo[at] = w64;
#pragma unroll
      for (int l = H64; l < O; ++l)
        out[((int64_t)m0 + (int64_t)l * a.ms - a.n_lo) * a.cells + at] = w[l];
    }
  }
  __syncthreads();                                  // before the next tile's loads
}

template <int K, int TIER>
__global__ __launch_bounds__(256) void colsweep_kernel(ColSweepArgs a) {
  extern __shared__ __align__(16) unsigned char colsweep_smem[];
  if (*as_ctab(a.flag) == 0) return;
  for (int32_t i = (int32_t)blockIdx.x; i < a.items; i += (int32_t)gridDim.x) {
    const int32_t w = (int32_t)xcd_tile((uint32_t)i, (uint32_t)a.items, 16);
    const uint32_t q1 = a.ftile.div((uint32_t)w);
    const int32_t tile = w - (int32_t)q1 * a.ntile;
    const int32_t spec = (int32_t)a.fQ.div(q1);
    const int32_t slab = (int32_t)q1 - spec * a.Q;
    const int32_t c0 = tile << a.logc;
    if (spec == 0 && a.n_lo == 1) {
      for (int32_t c = 0; c < 1 << a.logc; c += 1 << a.logc64)
        colsweep_tile<K, TIER, 1>(a, c0 + c, a.logc64, slab, spec, colsweep_smem);
    } else {
      colsweep_tile<K, TIER, 0>(a, c0, a.logc, slab, spec, colsweep_smem);
    }
  }
}

}  // namespace sldg
