// Fused pair of projection sweeps along two neighbouring dimensions d, d + 1 >= 1
// whose displacements depend only on the dimensions below d (L. Einkemmer,
// arXiv 1603.07008, section II: the split step's v1 and v2 sweeps, moved by
// E(x1, x2); section II-A update rule): one pass over the state, bitwise the
// two sweeps one after the other.
//
// Both sweeps act on a column (a cell of the dimensions below d) alone, with
// the column's own pair of shifts and matrices.  So a lane takes one column, 64
// neighbouring ones a wave, for one spectator group (the o^2 modes (j_d,
// j_{d+1})): it takes L rows of dimension d and walks R rows of dimension
// d + 1.  Per row of d + 1 it loads the L + 2 source rows of d (one row of d + 1
// ahead), applies the first sweep, rounds to the storage type as the separate
// sweep stores it, and keeps the result in registers for the second sweep, which
// reads the three latest rows.  No LDS for the state, no barrier in the walk;
// every access is 64 neighbouring cells at one row.
//
// L + 2 and three rows: a smooth field gives the 64 columns of a wave at most
// two neighbouring shifts per dimension (N - 1 and 0 around a zero of the
// field), and each lane picks its window of the rows loaded for the wave: whole
// rows instead of pieces of two (48^4, k = 2, FP32 840 us when every lane loads
// its own L + 1 rows, 745 so; bf16 577 and 433).  Waves with other shifts load
// each lane's own rows, scattered over both dimensions; fields of more than a few
// cells over a wave run the two sweeps by themselves instead (sldg_colsweep.h).
//
// Bound by memory: 48^4, k = 2 moves 3.4 GB in 732 us (4.8 TB/s; it reads 1.4 x
// the state: 10 rows of d per workgroup of 8, R + 2 of d + 1) where the two
// sweeps take 668 + 693; bf16 436 (416 + 415), FP16 461 (443 + 448), FP64 at 40^4
// 694 (643 + 691); k = 1 FP32 155 (140 + 150); 24^4, k = 3 FP32 203 (158 + 157).
// The registers set L: more rows or waves spill (k = 2 FP64 at two waves a SIMD:
// 1594 us; k = 3 with L = 2 there: 656).
#pragma once

#include "sldg_strang.h"

namespace sldg {

struct ColPairArgs {
  const double* in_lo;       // FP64 plane of mode 0 (n_lo == 1), or unused
  const void* in_hi;         // the other modes, storage type of the tier
  double* out_lo;
  void* out_hi;
  int32_t n_lo;
  int64_t cells;             // cells of the grid (plane length)
  int32_t P, N1, N2, Q;      // cells below d, extents of d and d + 1, cells above
  int32_t ms;                // o^d: mode-id stride of j_d (j_{d+1}: ms o)
  int32_t R, nstrip;         // rows of d + 1 per wave, strips
  int32_t nrow;              // waves along d: ceil(N1 / L)
  int32_t S, ngroup;         // strips whose waves fill whole workgroups, groups of S strips
  int32_t nblk;              // column blocks (64 columns) of a Q slab
  int32_t nchunk;            // workgroups of a column block and group: ceil(nrow S / 4)
  float one;                 // 1.0f: the FP16 tier's unit scale
  FastDiv fblk, fgroup, fchunk, fQ, frow;
  const int32_t* s1;         // the two sweeps' line tables, component-major
  const double* ab1;
  int64_t cs1;
  LineMap map1;
  const int32_t* s2;
  const double* ab2;
  int64_t cs2;
  LineMap map2;
  const int32_t* flag;       // the pass does nothing where *flag != 0 (may be null)
};

// Rows of dimension d per lane, and waves per SIMD (they bound the registers).
constexpr int colpair_rows(int k, int /*tier*/) { return k == 3 ? 1 : 2; }
constexpr int colpair_waves_per_simd(int k, int tier) { return k > 1 && tier == 0 ? 1 : 2; }

// The planes of one spectator group: mode (j_d, j_{d+1}) at `stride` (j_d + o
// j_{d+1}) bytes from the first, each its own buffer; a cell at the lane's byte
// offset plus a uniform one.
template <class T>
struct PairPlanes {
  const char* hi;
  const char* lo;
  int64_t stride;
  int32_t extent, extent64;

  __device__ __forceinline__ __amdgpu_buffer_rsrc_t plane(int m) const {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(hi) + m * stride, (short)0, extent,
                                             0x00020000);
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t plane64() const {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(lo), (short)0, extent64, 0x00020000);
  }
};

template <int K, int TIER, int H64>
struct PairIO {
  static constexpr int O = K + 1;
  using T = typename Tier<TIER>::T;
  using Cell = StrangCell<K, TIER, H64>;
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));

  // cell at the lane's offset (bytes: vt, v8 in the FP64 plane) and a uniform one so (cells)
  static __device__ __forceinline__ void load(const PairPlanes<T>& p, int32_t vt, int32_t v8,
                                              int32_t so, Cell& q) {
    if (H64)
      q.d = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(p.plane64(), v8, so * 8, 0));
#pragma unroll
    for (int l1 = 0; l1 < O; ++l1)
#pragma unroll
      for (int l0 = 0; l0 < O; ++l0) {
        if (H64 && l0 + l1 == 0) continue;
        const __amdgpu_buffer_rsrc_t r = p.plane(l0 + O * l1);
        const int32_t s = so * (int32_t)sizeof(T);
        if constexpr (sizeof(T) == 8)
          q.u[l1][l0] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, vt, s, 0));
        else if constexpr (sizeof(T) == 4)
          q.u[l1][l0] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, vt, s, 0));
        else
          q.u[l1][l0] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, vt, s, 0));
      }
  }
  // non-temporal: outputs are not read again
  static __device__ __forceinline__ void store(const PairPlanes<T>& p, int32_t vt, int32_t v8,
                                               int32_t so, const Cell& q) {
    if (H64)
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, q.d), p.plane64(), v8, so * 8, 2);
#pragma unroll
    for (int l1 = 0; l1 < O; ++l1)
#pragma unroll
      for (int l0 = 0; l0 < O; ++l0) {
        if (H64 && l0 + l1 == 0) continue;
        const __amdgpu_buffer_rsrc_t r = p.plane(l0 + O * l1);
        const int32_t s = so * (int32_t)sizeof(T);
        if constexpr (sizeof(T) == 8)
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, q.u[l1][l0]), r, vt, s, 2);
        else if constexpr (sizeof(T) == 4)
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, q.u[l1][l0]), r, vt, s, 2);
        else
          __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, q.u[l1][l0]), r, vt, s, 2);
      }
  }
  static __device__ __forceinline__ void pick(bool c, const Cell& a, const Cell& b, Cell& q) {
    if (H64) q.d = c ? a.d : b.d;
#pragma unroll
    for (int l1 = 0; l1 < O; ++l1)
#pragma unroll
      for (int l0 = 0; l0 < O; ++l0) q.u[l1][l0] = c ? a.u[l1][l0] : b.u[l1][l0];
  }
};

// The sweep along d of one cell (tuples (l, j1)) from source cells x, y.
template <int K, int TIER, int H64>
__device__ __forceinline__ void pair_first(float one, const Mat<K, TIER>& M,
                                           const Rows64<K, 1>& R64,
                                           const StrangCell<K, TIER, H64>& xc,
                                           const StrangCell<K, TIER, H64>& yc,
                                           StrangCell<K, TIER, H64>& w) {
  constexpr int O = K + 1;
  using T = typename Tier<TIER>::T;
#pragma unroll
  for (int l1 = 0; l1 < O; ++l1) {
    auto tuple = [&](auto ndc) {
      constexpr int ND = decltype(ndc)::value;
      Raw<K, TIER, ND> x, y;
#pragma unroll
      for (int l0 = 0; l0 < O; ++l0) {
        raw_set<K, TIER, ND>(x, l0, l0 < ND ? T(0) : xc.u[l1][l0], l0 < ND ? xc.d : 0.0, one);
        raw_set<K, TIER, ND>(y, l0, l0 < ND ? T(0) : yc.u[l1][l0], l0 < ND ? yc.d : 0.0, one);
      }
      strang_tuple<K, TIER, ND>(M, R64, x, y, w.u[l1], w.d, one);
    };
    if (H64 && l1 == 0) tuple(std::integral_constant<int, 1>{});
    else tuple(std::integral_constant<int, 0>{});
  }
}

// The matrices of the wave's columns in LDS (the workgroup's four waves share
// them): held in registers they would leave room for half the rows per lane.
// Component e of sweep i at lds[(i 2 o^2 + e) 64 + lane] in the arithmetic type,
// then for the 16-bit tiers the FP64 row 0 (A_0l, B_0l) of each sweep.
template <int K, int TIER>
struct PairMats {
  static constexpr int O = K + 1, O2 = O * O;
  using Acc = typename Tier<TIER>::Acc;
  static constexpr bool kRow64 = sizeof(Acc) == 4;
  Acc m[2][2 * O2][64];
  double r[kRow64 ? 2 : 1][kRow64 ? 2 * O : 1][kRow64 ? 64 : 1];

  __device__ __forceinline__ void fill(int i, const double* tab, int64_t cs, int32_t t, int lane,
                                       int wave) {
    const auto* ab = as_global(tab) + t;
    for (int e = wave; e < 2 * O2; e += 4) {
      const double v = ab[e * cs];
      m[i][e][lane] = (Acc)v;
      if constexpr (kRow64) {
        if (e < O) r[i][e][lane] = v;
        else if (e >= O2 && e < O2 + O) r[i][O + e - O2][lane] = v;
      }
    }
  }
  template <int H64>
  __device__ __forceinline__ void get(int i, int lane, Mat<K, TIER>& M, Rows64<K, 1>& R) const {
#pragma unroll
    for (int j = 0; j < O; ++j)
#pragma unroll
      for (int l = 0; l < O; ++l) {
        M.Aa[j][l] = m[i][j * O + l][lane];
        M.Ba[j][l] = m[i][O2 + j * O + l][lane];
        if (H64 && j == 0) {
          if constexpr (kRow64) {
            R.A[0][l] = r[i][l][lane];
            R.B[0][l] = r[i][O + l][lane];
          } else {
            R.A[0][l] = M.Aa[0][l];
            R.B[0][l] = M.Ba[0][l];
          }
        }
      }
  }
};

// Whether the wave's shifts s (in [0, N)) take at most two neighbouring values
// modulo N: lo is then the smaller one.
__device__ __forceinline__ bool two_shifts(int32_t s, int32_t N, int32_t& lo) {
  const int32_t s0 = __builtin_amdgcn_readfirstlane(s);
  const int32_t up = s0 + 1 == N ? 0 : s0 + 1, dn = s0 == 0 ? N - 1 : s0 - 1;
  const bool u = __all(s == s0 || s == up);
  lo = u ? s0 : dn;
  return u || __all(s == s0 || s == dn);
}

template <int K, int TIER, int H64>
__device__ __forceinline__ void colpair_body(const ColPairArgs& a, int32_t blk, int32_t chunk,
                                             int32_t strip, int32_t slab, int32_t g,
                                             PairMats<K, TIER>& mats) {
  constexpr int O = K + 1, L = colpair_rows(K, TIER);
  using T = typename Tier<TIER>::T;
  using Cell = StrangCell<K, TIER, H64>;
  using IO = PairIO<K, TIER, H64>;
  const int32_t P = a.P, N1 = a.N1, N2 = a.N2;
  const int32_t b1 = chunk * L;                     // first row of d
  const int32_t nrow = min(L, N1 - b1);
  const int32_t lane = (int32_t)(threadIdx.x & 63);
  const bool act = blk * 64 + lane < P;
  const int32_t col = min(blk * 64 + lane, P - 1);
  // spectator group g: g = low + ms * high, first mode low + ms o^2 high
  const int32_t low = g % a.ms, m0 = low + (g - low) * O * O;
  const int64_t sz = (int64_t)sizeof(T);
  PairPlanes<T> in, out;
  in.hi = reinterpret_cast<const char*>(a.in_hi) + (int64_t)(m0 - a.n_lo) * a.cells * sz;
  out.hi = reinterpret_cast<const char*>(a.out_hi) + (int64_t)(m0 - a.n_lo) * a.cells * sz;
  in.lo = reinterpret_cast<const char*>(a.in_lo);
  out.lo = reinterpret_cast<const char*>(a.out_lo);
  in.stride = out.stride = (int64_t)a.ms * a.cells * sz;
  in.extent = out.extent = (int32_t)(a.cells * sz);
  in.extent64 = out.extent64 = (int32_t)(a.cells * 8);

  const int32_t t1 = table_index(a.map1, col, 0), t2 = table_index(a.map2, col, 0);
  {
    const int wave = (int)(threadIdx.x >> 6);
    mats.fill(0, a.ab1, a.cs1, t1, lane, wave);
    mats.fill(1, a.ab2, a.cs2, t2, lane, wave);
  }
  __syncthreads();
  if (strip >= a.nstrip || (a.flag && *as_ctab(a.flag) != 0)) return;
  // a sweep's matrices, read again at each use
  auto get = [&](int i, Mat<K, TIER>& M, Rows64<K, 1>& R64) {
    asm volatile("" ::: "memory");
    mats.template get<H64>(i, lane, M, R64);
  };
  const int32_t s1 = as_global(a.s1)[t1], s2 = as_global(a.s2)[t2];
  const int32_t n1 = pin(N1), n2 = pin(N2), p = pin(P);
  const float one = pin(a.one);
  const int32_t base = slab * P * N1 * N2 + col;    // cells < 2^31 / 8
  const int32_t vt = base * (int32_t)sz, v8 = base * 8;
  const int32_t ot = act ? vt : INT32_MIN, o8 = act ? v8 : INT32_MIN;   // no store past the columns
  const int32_t r0 = strip * a.R, r1 = min(N2, r0 + a.R);
  const int32_t plane = n1 * p;
  struct Ring { Cell c[L]; };
  int32_t left;                                     // rows of d + 1 still to load
  // the planes to load from; empty past the last row: no memory is touched
  auto source = [&] {
    const bool live = --left >= 0;
    PairPlanes<T> src = in;
    src.extent = __builtin_amdgcn_readfirstlane(live ? in.extent : 0);
    src.extent64 = __builtin_amdgcn_readfirstlane(live ? in.extent64 : 0);
    return src;
  };
  // the second sweep of output row r from swept rows x (of the larger offset), y
  auto second = [&](int32_t r, bool up, const Ring& x0, const Ring& y0, const Ring& x1,
                    const Ring& y1) {
    const int32_t ro = r * plane + b1 * p;
    Mat<K, TIER> M2;
    Rows64<K, 1> R2;
    get(1, M2, R2);
#pragma unroll
    for (int u = 0; u < L; ++u) {
      Cell w;
      strang_v<K, TIER, H64>(one, M2, R2, up, x0.c[u], y0.c[u], x1.c[u], y1.c[u], w);
      // rows past the last one of d store past the buffer
      IO::store(out, u < nrow ? ot : INT32_MIN, u < nrow ? o8 : INT32_MIN, ro + u * p, w);
    }
  };

  int32_t lo1, lo2;
  if (two_shifts(s1, n1, lo1) & two_shifts(s2, n2, lo2)) {
    const bool up1 = s1 != lo1, up2 = s2 != lo2;
    // source rows of d: b1 - lo1 - 2 + v, v = 0 .. L + 1 (modulo N1)
    int32_t roff[L + 2];
    {
      int32_t i = b1 - lo1 - 2;
      while (i < 0) i += n1;
#pragma unroll
      for (int v = 0; v < L + 2; ++v) {
        roff[v] = i * p;
        i = i + 1 == n1 ? 0 : i + 1;
      }
    }
    // source row n of d + 1: r0 - lo2 - 2 + n (modulo N2)
    int32_t row = r0 - lo2 - 2;
    while (row < 0) row += n2;
    left = r1 - r0 + 2;
    struct Rows { Cell c[L + 2]; };
    Rows S;
    auto fetch = [&] {
      const PairPlanes<T> src = source();
      const int32_t ro = row * plane;
#pragma unroll
      for (int v = 0; v < L + 2; ++v) IO::load(src, vt, v8, ro + roff[v], S.c[v]);
      row = row + 1 == n2 ? 0 : row + 1;
    };
    // the first sweep of the fetched row
    auto first = [&](Ring& q) {
      Mat<K, TIER> M1;
      Rows64<K, 1> R1;
      get(0, M1, R1);
      Cell y;
      IO::pick(up1, S.c[0], S.c[1], y);
#pragma unroll
      for (int u = 0; u < L; ++u) {
        Cell x;
        IO::pick(up1, S.c[u + 1], S.c[u + 2], x);
        pair_first<K, TIER, H64>(one, M1, R1, x, y, q.c[u]);
        y = x;
      }
    };
    Ring q0, q1, q2;
    fetch();
    first(q0);
    fetch();
    first(q1);
    fetch();
    first(q2);
    fetch();
    auto step = [&](int32_t r, Ring& old, const Ring& mid, const Ring& neu) {
      second(r, up2, neu, mid, mid, old);
      first(old);
      fetch();
    };
    for (int32_t r = r0; r < r1; r += 3) {
      step(r, q0, q1, q2);
      if (r + 1 >= r1) break;
      step(r + 1, q1, q2, q0);
      if (r + 2 >= r1) break;
      step(r + 2, q2, q0, q1);
    }
    return;
  }

  // Spread shifts: byte offsets of the lane's own source rows of d, b1 - s1 - 1
  // + v (modulo N1), and its row of d + 1, r0 - s2 - 1 + n (modulo N2).
  int32_t rt[L + 1];
  {
    int32_t i = b1 - s1 - 1;
    i = i < 0 ? i + n1 : i;
#pragma unroll
    for (int v = 0; v < L + 1; ++v) {
      rt[v] = vt + i * p * (int32_t)sz;
      i = i + 1 == n1 ? 0 : i + 1;
    }
  }
  int32_t row = r0 - s2 - 1;
  row = row < 0 ? row + n2 : row;
  left = r1 - r0 + 1;
  struct Rows { Cell c[L + 1]; };
  Rows S;
  auto fetch = [&] {
    const PairPlanes<T> src = source();
    const int32_t ro = row * plane * (int32_t)sz;
#pragma unroll
    for (int v = 0; v < L + 1; ++v) {
      const int32_t o = rt[v] + ro;
      IO::load(src, o, o * (8 / (int32_t)sz), 0, S.c[v]);
    }
    row = row + 1 == n2 ? 0 : row + 1;
  };
  auto first = [&](Ring& q) {
    Mat<K, TIER> M1;
    Rows64<K, 1> R1;
    get(0, M1, R1);
#pragma unroll
    for (int u = 0; u < L; ++u)
      pair_first<K, TIER, H64>(one, M1, R1, S.c[u + 1], S.c[u], q.c[u]);
  };
  Ring q0, q1;
  fetch();
  first(q0);
  fetch();
  first(q1);
  fetch();
  auto step = [&](int32_t r, Ring& old, const Ring& cur) {
    second(r, false, cur, old, cur, old);
    first(old);
    fetch();
  };
  for (int32_t r = r0; r < r1; r += 2) {
    step(r, q0, q1);
    if (r + 1 >= r1) break;
    step(r + 1, q1, q0);
  }
}

template <int K, int TIER>
__global__ __launch_bounds__(256, colpair_waves_per_simd(K, TIER)) void sweep_colpair_kernel(
    ColPairArgs a) {
  // tile order: the workgroups along d of a column block first (they share
  // rows), then the column blocks, groups of strips, slabs and spectator groups.
  // The waves of a group of strips follow one another over the workgroups, so that
  // none is idle where four do not divide those along d.
  const uint32_t w = blockIdx.x;
  const uint32_t q1 = a.fchunk.div(w);
  const int32_t cg = (int32_t)(w - q1 * (uint32_t)a.nchunk);
  const uint32_t q2 = a.fblk.div(q1);
  const int32_t blk = (int32_t)(q1 - q2 * (uint32_t)a.nblk);
  const uint32_t q3 = a.fgroup.div(q2);
  const int32_t group = (int32_t)(q2 - q3 * (uint32_t)a.ngroup);
  const uint32_t g = a.fQ.div(q3);
  const int32_t slab = (int32_t)(q3 - g * (uint32_t)a.Q);
  const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
  const uint32_t task = (uint32_t)(cg * 4 + wave);
  const uint32_t of = a.frow.div(task);             // strip of the group (S: none)
  const int32_t chunk = (int32_t)(task - of * (uint32_t)a.nrow);
  const int32_t strip = of < (uint32_t)a.S ? group * a.S + (int32_t)of : a.nstrip;
  __shared__ PairMats<K, TIER> mats;
  if (g == 0 && a.n_lo == 1) colpair_body<K, TIER, 1>(a, blk, chunk, strip, slab, (int32_t)g, mats);
  else colpair_body<K, TIER, 0>(a, blk, chunk, strip, slab, (int32_t)g, mats);
}

}  // namespace sldg
