// Instantiation unit of the 1D split steps (sldg_line.h) for one degree k and
// one storage tier, selected when compiling (-DSLDG_K=1..3 -DSLDG_TIER=0..3) as
// sldg_sweep_inst.hip is.
#include "sldg_line.h"

#if !defined(SLDG_K) || !defined(SLDG_TIER)
#error "compile with -DSLDG_K=<degree> -DSLDG_TIER=<tier>"
#endif

namespace sldg {

template <int K, int TIER>
hipError_t launch_line_steps_inst(const LineStepsArgs& a, int cells, int32_t lds, hipStream_t st) {
  const int threads = ((a.N + cells - 1) / cells + 63) / 64 * 64;
  switch (cells) {
    case 1: line_steps_kernel<K, TIER, 1><<<1, threads, lds, st>>>(a); break;
    case 2: line_steps_kernel<K, TIER, 2><<<1, threads, lds, st>>>(a); break;
    case 4: line_steps_kernel<K, TIER, 4><<<1, threads, lds, st>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template hipError_t launch_line_steps_inst<SLDG_K, SLDG_TIER>(const LineStepsArgs&, int, int32_t,
                                                              hipStream_t);

}  // namespace sldg
