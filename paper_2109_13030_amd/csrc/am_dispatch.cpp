// am_dispatch.cpp -- picks the object of the fused kernel (one per element
// type and basis size) that serves a launch, and sizes its LDS.
#include "am_device.h"
#include "am_internal.h"

namespace amk {

template <typename T, int NV>
hipError_t launch_fused_part(const Desc &single, const Desc *table, int nprob, int nblocks, int max_m, hipStream_t st,
                             size_t lds_bytes, int tile, int waves);

size_t fused_lds_bytes(int q, int n, int nv, bool f64, int tile, int waves) {
  return size_t(fused_layout(q, n, nv, tile, red_rows_for(waves), f64 ? 1 : 2).total) * (f64 ? 8 : 4);
}

hipError_t launch_fused(const Desc &single, const Desc *table, int nprob, int nblocks, bool f64, int nv, int max_m,
                        hipStream_t st, size_t lds_bytes, int tile, int waves) {
  if (nblocks <= 0) return hipSuccess;
  if (max_m < 1 || max_m > AM_MAX_CIRCLES) return hipErrorInvalidValue;
  if (f64 && nv == 11)
    return launch_fused_part<double, 11>(single, table, nprob, nblocks, max_m, st, lds_bytes, tile, waves);
  if (f64 && nv == 8)
    return launch_fused_part<double, 8>(single, table, nprob, nblocks, max_m, st, lds_bytes, tile, waves);
  if (!f64 && nv == 11)
    return launch_fused_part<float, 11>(single, table, nprob, nblocks, max_m, st, lds_bytes, tile, waves);
  if (!f64 && nv == 8)
    return launch_fused_part<float, 8>(single, table, nprob, nblocks, max_m, st, lds_bytes, tile, waves);
  return hipErrorInvalidValue;
}

}  // namespace amk
