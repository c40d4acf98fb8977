// Instantiation unit of the fused X V X sweeps (sldg_strang.h) for one degree
// k and one storage tier, selected when compiling (-DSLDG_K=1..3
// -DSLDG_TIER=0..3) as sldg_sweep_inst.hip is.
#include "sldg_strang.h"

#if !defined(SLDG_K) || !defined(SLDG_TIER)
#error "compile with -DSLDG_K=<degree> -DSLDG_TIER=<tier>"
#endif

namespace sldg {

template <int K, int TIER>
hipError_t launch_strang_inst(int post, const StrangArgs& a, int32_t nblocks, hipStream_t st) {
  if (post == 1) sweep_strang_kernel<K, TIER, true, 1><<<nblocks, 64, 0, st>>>(a);
  else sweep_strang_kernel<K, TIER, false, 2><<<nblocks, 64, 0, st>>>(a);
  return hipGetLastError();
}

template <int K, int TIER>
hipError_t launch_batch_strang_inst(const StrangArgs* args, const BatchItem* items, int32_t nitems,
                                    int32_t xcd, hipStream_t st) {
  batch_strang_kernel<K, TIER><<<nitems, 64, 0, st>>>(args, items, xcd);
  return hipGetLastError();
}

template hipError_t launch_batch_strang_inst<SLDG_K, SLDG_TIER>(const StrangArgs*, const BatchItem*,
                                                                int32_t, int32_t, hipStream_t);
template hipError_t launch_strang_inst<SLDG_K, SLDG_TIER>(int, const StrangArgs&, int32_t,
                                                          hipStream_t);

}  // namespace sldg
