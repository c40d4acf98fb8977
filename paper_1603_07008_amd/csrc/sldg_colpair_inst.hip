// Instantiation unit of the fused column pair (sldg_colpair.h) and of its sweeps
// one by one (sldg_colsweep.h) for one degree k and one storage tier, selected when compiling (-DSLDG_K=1..3
// -DSLDG_TIER=0..3) as sldg_sweep_inst.hip is.
#include "sldg_colpair.h"
#include "sldg_colsweep.h"

#if !defined(SLDG_K) || !defined(SLDG_TIER)
#error "compile with -DSLDG_K=<degree> -DSLDG_TIER=<tier>"
#endif

namespace sldg {

template <int K, int TIER>
hipError_t launch_colpair_inst(const ColPairArgs& a, int32_t nblocks, hipStream_t st) {
  sweep_colpair_kernel<K, TIER><<<nblocks, 256, 0, st>>>(a);
  return hipGetLastError();
}

template <int K, int TIER>
hipError_t launch_colsweep_inst(const ColSweepArgs& a, int32_t nblocks, int32_t lds,
                                hipStream_t st) {
  colsweep_kernel<K, TIER><<<nblocks, 256, lds, st>>>(a);
  return hipGetLastError();
}

template hipError_t launch_colpair_inst<SLDG_K, SLDG_TIER>(const ColPairArgs&, int32_t, hipStream_t);
template hipError_t launch_colsweep_inst<SLDG_K, SLDG_TIER>(const ColSweepArgs&, int32_t, int32_t,
                                                            hipStream_t);

}  // namespace sldg
