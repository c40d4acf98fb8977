// Strang-fused sweeps of (x, v)-like slabs (L. Einkemmer, arXiv 1603.07008,
// section II: Cheng-Knorr splitting; section II-A update rule): consecutive
// sweeps along dimensions 0 and 1 as one pass over the state, bitwise the
// sweeps one after the other: X V X (PRE, POST = 1: a Strang step), or V X X
// (POST = 2: the end of one step and the start of the next where the field is
// solved for in between).  Unlike the fused pair of sldg_fused.h the
// displacements may vary as a split Vlasov step has them: those along
// dimension 0 from row to row (x moves with v), those along dimension 1 from
// column to column (v moves with E(x)), and by any number of cells.
//
// Every wave works on its own (no LDS, no barrier): it takes 64 columns of
// dimension 0, one per lane, of one slab (a fixed cell of the dimensions >= 2)
// and one spectator group (the o^2 modes (j0, j1)), and walks R rows of
// dimension 1.
//   X before V  a lane holds its column moved by the row's X shift (uniform
//               over the wave); its second source is the lane below's.
//   V           reads the lane's own column only, at rows r - s and r - s - 1
//               of the column's shift s: the X-swept rows stay in registers.
//               Where the wave's shifts take at most two neighbouring values
//               smin, smin + 1 (modulo N1), as a smooth field gives, row r
//               reads the X-swept rows r - smin, r - smin - 1, r - smin - 2:
//               each row is loaded (one row ahead) and X-swept once.  In
//               other waves each lane walks the rows of its own shift: it
//               X-sweeps its own cell of row r - s, loading that cell, its
//               lower neighbour's and the row's matrices itself.
//   X after V   again takes the second source from the lane below.
// The output cells of a row are the wave's columns moved by the row's X shifts:
// the columns, and the V matrices held for them, stay fixed while the outputs
// move, so no displacement needs a halo.  C + 2 lanes give C output cells.
// Every intermediate value is rounded to the storage type as the separate
// sweep stores it.
//
// Bound: one read and one write of the state for three sweeps; at k = 3 the
// FP64 arithmetic (384 multiply-adds per cell of a wave's row) is of the same
// size.  Keeping the rows in registers instead of LDS is what made it fast:
// the batched Landau workload's step took 2.33 ms sweep by sweep, 1.10 ms with
// the X-swept rows and the V-swept row in LDS (256 lanes, one barrier a row),
// 0.95 ms in this form.
// Waves of spread shifts load each X-swept cell's two sources (2 o^2 values) and
// the row's matrices per lane, whatever the number of shifts: a step of 512^2,
// k = 2, FP32, displacements to 3, 10 and 30 cells 15, 18 and 25 us (13 us to
// 1.5 cells; three sweeps 24), 256^2, k = 3, BF16 12, 14 and 20 (25-31); 2048^2,
// k = 2, FP32 106, 132 and 178 (222).  Evaluating both rows of every distinct
// shift of the wave took 19, 37 and 101 us on the first of these.  Slower than the
// sweeps: k = 3 at 512^2 and 30 cells, where a wave's lanes lie on some 24 rows
// (42 us against 35).
#pragma once

#include "sldg_fused.h"

namespace sldg {

// One sweep's line table: component e of entry t at ab[e * cs + t * ts].  The
// entry of a line is base + step * i, i the row (X sweeps) or column (V) and
// base that of the slab (`map`, over the dimensions above; step 0 where the
// displacement does not vary along i).  The X tables are entry-major (cs 1),
// so that a row's matrices are one run of scalar loads; the V table is
// component-major (ts 1), so that neighbouring columns read neighbouring
// addresses.
struct LineTable {
  const int32_t* s;
  const double* ab;
  int64_t cs, ts;
  int32_t step;
  LineMap map;
};

struct StrangArgs {
  const double* in_lo;       // FP64 plane of mode 0 (n_lo == 1), or unused
  const void* in_hi;         // the other modes, storage type of the tier
  double* out_lo;
  void* out_hi;
  int32_t n_lo;              // 1: mode 0 stored in FP64; 0: every mode narrow
  int64_t cells;             // cells of the grid (plane length)
  int32_t N0, N1;            // extents of dimensions 0 and 1
  int32_t Q;                 // slabs
  int32_t C;                 // output cells of dimension 0 per tile
  int32_t ntile;             // ceil(N0 / C)
  int32_t R;                 // rows per wave (at most kStrangMaxRows)
  int32_t nstrip;            // ceil(N1 / R)
  int32_t xcd;               // XCD-aware tile order: run length G (0 off)
  float one;                 // 1.0f: the FP16 tier's unit scale (see tuple4 in sldg_fused.h)
  FastDiv fstrip, ftile, fQ;
  LineTable x0, v, x1;       // the X sweep before V, V, the X sweep(s) after V
};

// Whether the planes of a spectator group fit 31-bit byte offsets.
inline bool strang_fits(int64_t cells, int64_t o, int64_t size) {
  return o * o * cells * size <= (int64_t)INT32_MAX && cells * 8 <= (int64_t)INT32_MAX;
}

// Whether a pass over grids of `lines` wave rows in all pays for lines of N0
// cells: its tiles take 64 lanes whatever their cells, so short lines leave lanes
// idle, which costs where the chip is full.  Measured (smooth displacements, a
// step as a pass and as three sweeps): 4 x 1024 x 64, k = 2, FP32 118 and 47 us, 8
// cells 64 and 44, 16 cells 38 and 43; k = 3, BF16 16 cells 97 and 61, 20 cells 84
// and 65, 24 cells 85 and 89; k = 1, BF16 8 cells 22 and 20; FP64 at k = 3 8 cells
// 263 and 156, 16 cells 142 and 169.  Small grids wait for launches instead (4 x
// 4096, k = 3, FP32: 14 us and 27).
constexpr int64_t kStrangFull = 16384;
inline bool strang_pays(int k, int64_t size, int64_t N0, int64_t lines) {
  const int64_t nt = (N0 + 61) / 62, C = (N0 + nt - 1) / nt;
  return lines < kStrangFull || C >= (size == 8 ? 4 * k + 4 : k == 1 ? 12 : k == 2 ? 20 : 24);
}

constexpr int kStrangMaxRows = 60;        // a strip's shifts (R + 4 rows) in one wave's lanes

// Tiles of dimension 0: the fewest of at most 62 cells; strips of `rows` rows.
inline void strang_tiles(StrangArgs& a, int32_t rows) {
  const int32_t nt = (a.N0 + 61) / 62;
  a.C = (a.N0 + nt - 1) / nt;
  a.ntile = (a.N0 + a.C - 1) / a.C;
  const int32_t ns = (a.N1 + rows - 1) / rows;
  a.R = (a.N1 + ns - 1) / ns;
  a.nstrip = (a.N1 + a.R - 1) / a.R;
}

// Waves per SIMD the kernels are compiled for (their registers: 256 for FP32
// at k = 3, 128 at k = 2, 80 at k = 1; 16-bit k = 3 takes 217, and at three
// waves it spills, 2048^2 190 us a step against 138).
constexpr int strang_waves_per_simd(int k, int tier) {
  return k == 3 ? (tier == 0 ? 1 : 2) : k == 2 ? (tier == 0 ? 3 : 4) : 6;
}

// Tables at wave-uniform entries, read through the constant address space:
// they were written by an earlier kernel, and without it the compiler must
// take the row loop's stores for possible writes to them and reads them with
// vector loads.
template <class T>
using ctab = const __attribute__((address_space(4))) T*;
template <class T>
__device__ __forceinline__ ctab<T> as_ctab(const T* p) {
  return (ctab<T>)(uintptr_t)p;
}

// A pointer read from an argument block, as one to global memory.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(1))) T* as_global(const T* p) {
  return (const __attribute__((address_space(1))) T*)(uintptr_t)p;
}

// The matrices of entry t of an entry-major line table, the same in every
// lane.
template <int K, int TIER, int H64>
__device__ __forceinline__ void load_uniform(ctab<double> tab, int32_t t, Mat<K, TIER>& M,
                                             Rows64<K, 1>& R) {
  constexpr int O = K + 1;
  const ctab<double> ab = tab + (int64_t)t * (2 * O * O);
#pragma unroll
  for (int j = 0; j < O; ++j)
#pragma unroll
    for (int l = 0; l < O; ++l) {
      const double A = ab[j * O + l], B = ab[O * O + j * O + l];
      M.Aa[j][l] = (typename Tier<TIER>::Acc)A;
      M.Ba[j][l] = (typename Tier<TIER>::Acc)B;
      if (H64 && j == 0) {
        R.A[0][l] = A;
        R.B[0][l] = B;
      }
    }
}

// The planes of one spectator group over one slab, as buffers: plane l at byte
// offset l * cells * size (a scalar) from the group's plane 0, cells at 32-bit
// byte offsets in vector registers (the host keeps a group's planes below 2^31
// bytes).  Plain pointers would take a 64-bit vector addition per access, and
// those read from an argument block in memory would be accessed through the
// flat address space, whose loads also hold up every wait for LDS.
template <class T>
struct GroupPlanes {
  __amdgpu_buffer_rsrc_t hi, lo;
  int32_t pstride;                             // bytes from plane to plane

  __device__ __forceinline__ void bind(const void* h, const double* l, int64_t hi_off,
                                       int64_t lo_off, int64_t cells, int o2) {
    constexpr int32_t kFlags = 0x00020000;     // raw buffer, 32-bit data format
    const T* p = reinterpret_cast<const T*>(h) + hi_off;
    hi = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), (short)0,
                                           (int32_t)(o2 * cells * (int64_t)sizeof(T)), kFlags);
    lo = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(l + lo_off), (short)0,
                                           (int32_t)(cells * 8), kFlags);
    pstride = (int32_t)(cells * (int64_t)sizeof(T));
  }
  __device__ __forceinline__ double get64(uint32_t c) const {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(lo, (int32_t)(c * 8u), 0, 0));
  }
  __device__ __forceinline__ T get(int l, uint32_t c) const {
    const int32_t v = (int32_t)(c * (uint32_t)sizeof(T)), so = l * pstride;
    if constexpr (sizeof(T) == 8)
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(hi, v, so, 0));
    else if constexpr (sizeof(T) == 4)
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(hi, v, so, 0));
    else
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(hi, v, so, 0));
  }
  // Stores at the byte offsets of cell c (`at`, `at64`).  A lane without a
  // cell stores at 2^31, past every plane, which writes nothing: no branch
  // splits the code around the stores.
  static __device__ __forceinline__ int32_t at(uint32_t c, bool live) {
    return live ? (int32_t)(c * (uint32_t)sizeof(T)) : INT32_MIN;
  }
  static __device__ __forceinline__ int32_t at64(uint32_t c, bool live) {
    return live ? (int32_t)(c * 8u) : INT32_MIN;
  }
  __device__ __forceinline__ void put64(int32_t v, double x) const {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, x), lo, v, 0, 0);
  }
  __device__ __forceinline__ void put(int l, int32_t v, T x) const {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    const int32_t so = l * pstride;
    if constexpr (sizeof(T) == 8)
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, x), hi, v, so, 0);
    else if constexpr (sizeof(T) == 4)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), hi, v, so, 0);
    else
      __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, x), hi, v, so, 0);
  }
};

// The outputs of one tuple from its two source cells, rounded to the storage
// type as the separate sweep stores them: out64 is the FP64 mode's (ND == 1).
template <int K, int TIER, int ND>
__device__ __forceinline__ void strang_tuple(const Mat<K, TIER>& M, const Rows64<K, 1>& R64,
                                             const Raw<K, TIER, ND>& x, const Raw<K, TIER, ND>& y,
                                             typename Tier<TIER>::T (&out)[K + 1], double& out64,
                                             float one) {
  using T = typename Tier<TIER>::T;
#pragma unroll
  for (int j = 0; j < K + 1; ++j) {
    if (j < ND) {
      Rows64<K, ND> r;
#pragma unroll
      for (int l = 0; l < K + 1; ++l) {
        r.A[0][l] = R64.A[0][l];
        r.B[0][l] = R64.B[0][l];
      }
      out64 = Mat<K, TIER>::template out64<ND>(r, 0, x, y);
    } else if constexpr (TIER == 3) {
      out[j] = (T)(M.template out_acc<ND>(j, x, y) * one);
    } else {
      out[j] = narrow<T>(M.template out_acc<ND>(j, x, y));
    }
  }
}

// The value of the lane below (lane 0: its own).
template <class T>
__device__ __forceinline__ T lane_below(T v) {
  if constexpr (sizeof(T) == 8) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = lane_below((uint32_t)b), hi = lane_below((uint32_t)(b >> 32));
    return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
  } else if constexpr (sizeof(T) == 2) {
    return __builtin_bit_cast(T, (uint16_t)lane_below((uint32_t)__builtin_bit_cast(uint16_t, v)));
  } else {
    const int b = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(b, b, 0x138, 0xF, 0xF, false));  // wave_shr 1
  }
}

// A uniform value the compiler must keep (it may otherwise read it from memory
// again at each use).
template <class V>
__device__ __forceinline__ V pin(V v) {
  asm volatile("" : "+s"(v));
  return v;
}

// A column of one row, [l1][l0], and mode (0, 0) where it is FP64: as stored,
// or after a sweep (rounded to the storage type).
template <int K, int TIER, int H64>
struct StrangCell {
  static constexpr int O = K + 1;
  using T = typename Tier<TIER>::T;
  T u[O][O];
  double d;

  __device__ __forceinline__ void load(const GroupPlanes<T>& in, uint32_t c) {
    if (H64) d = in.get64(c);
#pragma unroll
    for (int l1 = 0; l1 < O; ++l1)
#pragma unroll
      for (int l0 = 0; l0 < O; ++l0)
        if (!(H64 && l0 + l1 == 0)) u[l1][l0] = in.get(l0 + O * l1, c);
  }
};

// The X sweep of a row in place: the lane's own source is its cell q, the other
// one y, or the lane below's where y is q itself.
template <int K, int TIER, int H64>
__device__ __forceinline__ void strang_x(float one, const Mat<K, TIER>& M,
                                         const Rows64<K, 1>& R64, StrangCell<K, TIER, H64>& q,
                                         const StrangCell<K, TIER, H64>* yc = nullptr) {
  constexpr int O = K + 1;
  using T = typename Tier<TIER>::T;
#pragma unroll
  for (int l1 = 0; l1 < O; ++l1) {
    auto tuple = [&](auto ndc) {
      constexpr int ND = decltype(ndc)::value;
      Raw<K, TIER, ND> x, y;
#pragma unroll
      for (int l0 = 0; l0 < O; ++l0) {
        raw_set<K, TIER, ND>(x, l0, l0 < ND ? T(0) : q.u[l1][l0], l0 < ND ? q.d : 0.0, one);
        raw_set<K, TIER, ND>(y, l0, l0 < ND ? T(0) : yc ? yc->u[l1][l0] : lane_below(q.u[l1][l0]),
                             l0 < ND ? (yc ? yc->d : lane_below(q.d)) : 0.0, one);
      }
      strang_tuple<K, TIER, ND>(M, R64, x, y, q.u[l1], q.d, one);
    };
    if (H64 && l1 == 0) tuple(std::integral_constant<int, 1>{});
    else tuple(std::integral_constant<int, 0>{});
  }
}

// The V sweep of a column from its two source cells (x through A, y through
// B): narrow outputs in w.u[j1][j0].  PICK: the sources are (x1, y1) where
// `second`, else (x0, y0).
template <int K, int TIER, int H64>
__device__ __forceinline__ void strang_v(float one, const Mat<K, TIER>& M, const Rows64<K, 1>& R64,
                                         bool second, const StrangCell<K, TIER, H64>& x0,
                                         const StrangCell<K, TIER, H64>& y0,
                                         const StrangCell<K, TIER, H64>& x1,
                                         const StrangCell<K, TIER, H64>& y1,
                                         StrangCell<K, TIER, H64>& w) {
  constexpr int O = K + 1;
  using T = typename Tier<TIER>::T;
#pragma unroll
  for (int j0 = 0; j0 < O; ++j0) {
    auto tuple = [&](auto ndc) {
      constexpr int ND = decltype(ndc)::value;
      Raw<K, TIER, ND> x, y;
#pragma unroll
      for (int l = 0; l < O; ++l) {
        const T xv = second ? x1.u[l][j0] : x0.u[l][j0];
        const T yv = second ? y1.u[l][j0] : y0.u[l][j0];
        raw_set<K, TIER, ND>(x, l, l < ND ? T(0) : xv, l < ND ? (second ? x1.d : x0.d) : 0.0, one);
        raw_set<K, TIER, ND>(y, l, l < ND ? T(0) : yv, l < ND ? (second ? y1.d : y0.d) : 0.0, one);
      }
      T o[O];
      strang_tuple<K, TIER, ND>(M, R64, x, y, o, w.d, one);
#pragma unroll
      for (int j1 = ND; j1 < O; ++j1) w.u[j1][j0] = o[j1];
    };
    if (H64 && j0 == 0) tuple(std::integral_constant<int, 1>{});
    else tuple(std::integral_constant<int, 0>{});
  }
}

template <int K, int TIER, bool PRE, int POST, int H64>
__device__ __forceinline__ void strang_body(const StrangArgs& a, int32_t tile, int32_t strip,
                                            int32_t slab, int32_t g) {
  constexpr int O = K + 1, O2 = O * O;
  using T = typename Tier<TIER>::T;
  using Cell = StrangCell<K, TIER, H64>;
  const int32_t N0 = a.N0, N1 = a.N1;
  const int32_t c0 = tile * a.C, nout = min(a.C, N0 - c0);
  const int32_t c = (int32_t)threadIdx.x;
  const bool act = c > 1 && c <= nout + 1;          // the lane has an output cell
  int32_t col = c0 + min(c, nout + 1);
  while (col >= N0) col -= N0;
  const int32_t r0 = strip * a.R, r1 = min(N1, r0 + a.R);

  const int64_t slab_off = (int64_t)slab * N1 * N0;
  const int64_t goff = ((int64_t)g * O2 - a.n_lo) * a.cells + slab_off;
  GroupPlanes<T> in, out;
  in.bind(a.in_hi, a.in_lo, goff, slab_off, a.cells, O2);
  out.bind(a.out_hi, a.out_lo, goff, slab_off, a.cells, O2);

  // the column's V shift and matrices
  Mat<K, TIER> MV;
  Rows64<K, 1> RV;
  const int32_t tv = table_index(a.v.map, 0, slab) + a.v.step * col;
  const int32_t sv = as_global(a.v.s)[tv];
  {
    const auto* ab = as_global(a.v.ab) + tv;
#pragma unroll
    for (int j = 0; j < O; ++j)
#pragma unroll
      for (int l = 0; l < O; ++l) {
        const double A = ab[(j * O + l) * a.v.cs], B = ab[(O2 + j * O + l) * a.v.cs];
        MV.Aa[j][l] = (typename Tier<TIER>::Acc)A;
        MV.Ba[j][l] = (typename Tier<TIER>::Acc)B;
        if (H64 && j == 0) {
          RV.A[0][l] = A;
          RV.B[0][l] = B;
        }
      }
  }

  // Uniform values the row loop reads, kept in scalar registers (read from the
  // argument block each time, they would put a memory latency in the loop).
  const int32_t n0 = pin(N0), n1 = pin(N1);
  const int32_t tb0 = PRE ? table_index(a.x0.map, 0, N1 * slab) : 0;
  const int32_t tb1 = table_index(a.x1.map, 0, N1 * slab);
  const ctab<double> ab0 = pin(as_ctab(a.x0.ab) + (int64_t)tb0 * (2 * O2));
  const ctab<double> ab1 = pin(as_ctab(a.x1.ab) + (int64_t)tb1 * (2 * O2));
  const int32_t step0 = pin(a.x0.step), step1 = pin(a.x1.step);
  const float one = pin(a.one);

  // a row's cells, moved by the X shift s where an X sweep comes first
  auto fetch = [&](Cell& q, int32_t row, int32_t s) {
    int32_t ix = col;
    if constexpr (PRE) {
      ix -= s;
      if (ix < 0) ix += n0;
    }
    q.load(in, (uint32_t)row * (uint32_t)n0 + (uint32_t)ix);
  };
  auto mats0 = [&](int32_t row, Mat<K, TIER>& M, Rows64<K, 1>& R64) {
    if constexpr (PRE) load_uniform<K, TIER, H64>(ab0, step0 * row, M, R64);
  };
  // the X sweeps after V of row r (matrices M, shift s), and the stores
  auto finish = [&](int32_t r, int32_t s, const Mat<K, TIER>& M, const Rows64<K, 1>& R64, Cell& w) {
#pragma unroll
    for (int q = 0; q < POST; ++q) strang_x<K, TIER, H64>(one, M, R64, w);
    int32_t oc = col;
#pragma unroll
    for (int q = 0; q < POST; ++q) {
      oc += s;
      if (oc >= n0) oc -= n0;
    }
    const uint32_t cell = (uint32_t)r * (uint32_t)n0 + (uint32_t)oc;
    const int32_t vo = out.at(cell, act), v8 = out.at64(cell, act);
    if (H64) out.put64(v8, w.d);
#pragma unroll
    for (int l1 = 0; l1 < O; ++l1)
#pragma unroll
      for (int l0 = 0; l0 < O; ++l0)
        if (!(H64 && l0 + l1 == 0)) out.put(l0 + O * l1, vo, w.u[l1][l0]);
  };
  // lane i: the shift of the X sweep after V for row r0 + i
  const int32_t sp = as_global(a.x1.s)[tb1 + step1 * min(r0 + c, N1 - 1)];

  auto next_row = [&](int32_t q) { return q + 1 == n1 ? 0 : q + 1; };
  const int32_t s0 = __builtin_amdgcn_readfirstlane(sv);
  const int32_t up = s0 + 1 == n1 ? 0 : s0 + 1, dn = s0 == 0 ? n1 - 1 : s0 - 1;
  const bool two_up = __all(sv == s0 || sv == up);
  if (!two_up && !__all(sv == s0 || sv == dn)) {
    // shifts all over: every lane walks the source rows of its own shift, and
    // X-sweeps its own cell of them, from that cell and its lower neighbour's
    int32_t row = r0 - sv - 1;
    if (row < 0) row += n1;
    int32_t sn = PRE ? as_global(a.x0.s)[tb0 + step0 * row] : 0;
    Cell S, Y;                                      // the cells of row `row`
    int32_t at = 0;                                 // ... and its table entry
    auto gather = [&] {
      const uint32_t line = (uint32_t)row * (uint32_t)n0;
      int32_t ix = col;
      if constexpr (PRE) {
        ix -= sn;
        if (ix < 0) ix += n0;
        Y.load(in, line + (uint32_t)(ix == 0 ? n0 - 1 : ix - 1));
        at = tb0 + step0 * row;
      }
      S.load(in, line + (uint32_t)ix);
      row = next_row(row);
      if constexpr (PRE) sn = as_global(a.x0.s)[tb0 + step0 * row];
    };
    auto swept = [&](Cell& q) {
      if constexpr (PRE) {
        Mat<K, TIER> M;
        Rows64<K, 1> R64;
        const auto* ab = as_global(a.x0.ab) + (int64_t)at * (2 * O2);
#pragma unroll
        for (int j = 0; j < O; ++j)
#pragma unroll
          for (int l = 0; l < O; ++l) {
            const double A = ab[j * O + l], B = ab[O2 + j * O + l];
            M.Aa[j][l] = (typename Tier<TIER>::Acc)A;
            M.Ba[j][l] = (typename Tier<TIER>::Acc)B;
            if (H64 && j == 0) {
              R64.A[0][l] = A;
              R64.B[0][l] = B;
            }
          }
        strang_x<K, TIER, H64>(one, M, R64, S, &Y);
      }
      q = S;
    };
    Cell old, cur;
    gather();
    swept(old);
    gather();
    swept(cur);
    gather();
    auto step = [&](int32_t r, Cell& o, const Cell& c) {
      Mat<K, TIER> M1;
      Rows64<K, 1> R1;
      load_uniform<K, TIER, H64>(ab1, step1 * r, M1, R1);
      Cell w;
      strang_v<K, TIER, H64>(one, MV, RV, false, c, o, c, o, w);
      finish(r, __builtin_amdgcn_readlane(sp, r - r0), M1, R1, w);
      swept(o);
      gather();
    };
    for (int32_t r = r0; r < r1; r += 2) {
      step(r, old, cur);
      if (r + 1 >= r1) break;
      step(r + 1, cur, old);
    }
    return;
  }
  const int32_t smin = two_up ? s0 : dn;
  const bool second = sv != smin;

  // Row n of the strip's sources is row r0 - smin - 2 + n (modulo N1); lane n
  // holds its X shift.
  int32_t row = r0 - smin - 2;
  while (row < 0) row += n1;
  const int32_t sx = PRE ? as_global(a.x0.s)[tb0 + step0 * ((row + c) % N1)] : 0;
  const int32_t row1 = next_row(row), row2 = next_row(row1);
  Cell q0, q1, q2, S;
  fetch(q0, row, __builtin_amdgcn_readlane(sx, 0));
  fetch(q1, row1, __builtin_amdgcn_readlane(sx, 1));
  fetch(q2, row2, __builtin_amdgcn_readlane(sx, 2));
  if constexpr (PRE) {
    Mat<K, TIER> M;
    Rows64<K, 1> R64;
    mats0(row, M, R64);
    strang_x<K, TIER, H64>(one, M, R64, q0);
    mats0(row1, M, R64);
    strang_x<K, TIER, H64>(one, M, R64, q1);
    mats0(row2, M, R64);
    strang_x<K, TIER, H64>(one, M, R64, q2);
  }
  row = next_row(row2);
  int32_t n = 3;
  fetch(S, row, __builtin_amdgcn_readlane(sx, 3));

  // row r from the source rows (oldest, middle, newest); the next one takes
  // the oldest one's place.  The matrices of both X sweeps are loaded before
  // the V sweep where the scalar registers hold them (k <= 2).
  auto step = [&](int32_t r, Cell& old, const Cell& mid, const Cell& neu) {
    Mat<K, TIER> M0, M1;
    Rows64<K, 1> R0, R1;
    load_uniform<K, TIER, H64>(ab1, step1 * r, M1, R1);
    if constexpr (K <= 2) mats0(row, M0, R0);
    Cell w;
    strang_v<K, TIER, H64>(one, MV, RV, second, neu, mid, mid, old, w);
    finish(r, __builtin_amdgcn_readlane(sp, r - r0), M1, R1, w);
    if constexpr (K > 2) mats0(row, M0, R0);
    if constexpr (PRE) strang_x<K, TIER, H64>(one, M0, R0, S);
    old = S;
    row = next_row(row);
    ++n;
    fetch(S, row, __builtin_amdgcn_readlane(sx, n));
  };
  for (int32_t r = r0; r < r1; r += 3) {
    step(r, q0, q1, q2);
    if (r + 1 >= r1) break;
    step(r + 1, q1, q2, q0);
    if (r + 2 >= r1) break;
    step(r + 2, q2, q0, q1);
  }
}

template <int K, int TIER, bool PRE, int POST>
__device__ __forceinline__ void strang_tile(const StrangArgs& a, int32_t tile, int32_t strip,
                                            int32_t slab, int32_t g) {
  if (g == 0 && a.n_lo == 1) strang_body<K, TIER, PRE, POST, 1>(a, tile, strip, slab, g);
  else strang_body<K, TIER, PRE, POST, 0>(a, tile, strip, slab, g);
}

template <int K, int TIER, bool PRE, int POST>
__global__ __launch_bounds__(64, strang_waves_per_simd(K, TIER)) void sweep_strang_kernel(
    StrangArgs a) {
  // tile order: the tiles of a strip first (they share cache lines)
  const uint32_t w = xcd_tile(blockIdx.x, gridDim.x, a.xcd);
  const uint32_t q1 = a.ftile.div(w);
  const int32_t tile = (int32_t)(w - q1 * (uint32_t)a.ntile);
  const uint32_t q2 = a.fstrip.div(q1);
  const int32_t strip = (int32_t)(q1 - q2 * (uint32_t)a.nstrip);
  const uint32_t g = a.fQ.div(q2);
  const int32_t slab = (int32_t)(q2 - g * (uint32_t)a.Q);
  strang_tile<K, TIER, PRE, POST>(a, tile, strip, slab, (int32_t)g);
}

// X V X of a batch: one wave per item (kind: tile, x: strip, z: slab, qg:
// spectator group) of one degree.
template <int K, int TIER>
__global__ __launch_bounds__(64, strang_waves_per_simd(K, TIER)) void batch_strang_kernel(
    const StrangArgs* __restrict__ args, const BatchItem* __restrict__ items, int32_t xcd) {
  const BatchItem w = items[xcd_tile(blockIdx.x, gridDim.x, xcd)];
  strang_tile<K, TIER, true, 1>(args[w.prob], w.kind, w.x, w.z, w.qg);
}

}  // namespace sldg
