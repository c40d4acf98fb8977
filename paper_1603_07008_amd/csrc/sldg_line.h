// The split steps of a 1D problem (the advection study of L. Einkemmer, arXiv
// 1603.07008, section III; section II-A update rule): many sweeps of one line in
// one launch, bitwise the sweeps one by one.
//
// A line of up to a few thousand cells fits the LDS of one compute unit, so one
// workgroup keeps it there from the first sweep to the last: per sweep a lane
// reads its cells' two sources, computes, rounds to the storage type as the
// separate sweep stores it, and writes its cells back.  Two copies of the line
// alternate, with one barrier a sweep, where LDS has room; else the line is
// updated in place between two barriers.
//
// Bound by the latency of a sweep's chain (LDS read, 2 o dependent FMAs, LDS
// write, barrier): 0.2 us a sweep at 64 cells, k = 2, FP64, 1.3 us at 4096 (the
// LDS traffic of one compute unit), where a launch a sweep takes 3.8 us with its
// gap.
#pragma once

#include "sldg_strang.h"

namespace sldg {

struct LineStepsArgs {
  const double* in_lo;       // FP64 plane of mode 0 (n_lo == 1), or unused
  const void* in_hi;         // the other modes, storage type of the tier
  double* out_lo;
  void* out_hi;
  int32_t n_lo, N;
  int32_t nseq, sweeps;      // sweeps of the sequence, sweeps of this launch
  int32_t stride;            // bytes from one copy of the line in LDS to the other (0: in place)
  float one;                 // 1.0f: the FP16 tier's unit scale
  const int32_t* s;          // line tables: entry pre[q] of sweep q
  const double* ab;
  int32_t pre[kMaxTableSet];
};

// Bytes of a cell.
constexpr int64_t line_cell_bytes(int o, int64_t n_lo, int64_t elem) {
  return 8 * n_lo + (o - n_lo) * elem;
}

// C cells per lane.
template <int K, int TIER, int C, int H64>
__device__ __forceinline__ void line_steps_body(const LineStepsArgs& a, unsigned char* smem) {
  constexpr int O = K + 1;
  using T = typename Tier<TIER>::T;
  const int32_t N = a.N, lane = (int32_t)threadIdx.x, step = (int32_t)blockDim.x;
  auto d = [&](int32_t b) { return reinterpret_cast<double*>(smem + b); };
  auto u = [&](int32_t b, int l) {
    return reinterpret_cast<T*>(smem + b + (H64 ? 8 * N : 0)) + (l - H64) * N;
  };
  for (int32_t c = lane; c < N; c += step) {
    if (H64) d(0)[c] = as_global(a.in_lo)[c];
    for (int l = H64; l < O; ++l)
      u(0, l)[c] = as_global(reinterpret_cast<const T*>(a.in_hi))[(int64_t)(l - H64) * N + c];
  }
  __syncthreads();
  const ctab<double> ab = as_ctab(a.ab);
  Mat<K, TIER> M;
  Rows64<K, 1> R;
  int32_t s = 0, q = 0, b = 0;
  for (int32_t n = 0; n < a.sweeps; ++n) {
    if (n == 0 || a.nseq > 1) {
      s = as_ctab(a.s)[a.pre[q]];
      load_uniform<K, TIER, H64>(ab, a.pre[q], M, R);
    }
    q = q + 1 == a.nseq ? 0 : q + 1;
    T w[C][O];
    double w64[C];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const int32_t c = min(lane + i * step, N - 1);
      int32_t j = c - s;
      j = j < 0 ? j + N : j;
      const int32_t j1 = j == 0 ? N - 1 : j - 1;
      Raw<K, TIER, H64> x, y;
#pragma unroll
      for (int l = 0; l < O; ++l) {
        raw_set<K, TIER, H64>(x, l, l < H64 ? T(0) : u(b, l)[j], l < H64 ? d(b)[j] : 0.0, a.one);
        raw_set<K, TIER, H64>(y, l, l < H64 ? T(0) : u(b, l)[j1], l < H64 ? d(b)[j1] : 0.0, a.one);
      }
      strang_tuple<K, TIER, H64>(M, R, x, y, w[i], w64[i], a.one);
    }
    if (a.stride == 0) __syncthreads();               // every source is read
    b = a.stride - b;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const int32_t c = lane + i * step;
      if (c < N) {
        if (H64) d(b)[c] = w64[i];
#pragma unroll
        for (int l = H64; l < O; ++l) u(b, l)[c] = w[i][l];
      }
    }
    __syncthreads();
  }
  for (int32_t c = lane; c < N; c += step) {
    if (H64) a.out_lo[c] = d(b)[c];
    for (int l = H64; l < O; ++l)
      reinterpret_cast<T*>(a.out_hi)[(int64_t)(l - H64) * N + c] = u(b, l)[c];
  }
}

template <int K, int TIER, int C>
__global__ __launch_bounds__(1024) void line_steps_kernel(LineStepsArgs a) {
  extern __shared__ __align__(16) unsigned char line_smem[];
  if (a.n_lo == 1) line_steps_body<K, TIER, C, 1>(a, line_smem);
  else line_steps_body<K, TIER, C, 0>(a, line_smem);
}

}  // namespace sldg
