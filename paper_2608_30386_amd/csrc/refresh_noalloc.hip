// dasc_refresh_noalloc: the bounded-suffix refresh of dasc_refresh for callers that
// cannot allocate device memory (code under HIP graph capture, tight serving loops,
// harnesses that forbid hipMalloc).
//
// No refresh kernel uses device scratch: every chunk's factors live in LDS.  What is left here
// is the limit the interface states (DASC_NOALLOC_SCRATCH_BYTES), kept so that the same
// requests are taken and refused.

#include <hip/hip_runtime.h>

#include <cstdint>

#include "dasc.h"
#include "dasc_testing.h"
#include "launch_common.h"
#include "refresh_kernels.h"

extern "C" int dasc_refresh_noalloc(const dasc_shape* shape, int32_t layer,
                                    const int32_t* inv_row, float* states, int64_t n_pool,
                                    const int32_t* slot, const uint16_t* k, const uint16_t* v,
                                    const float* g, const float* beta, int32_t n_req, int32_t W,
                                    int32_t init_mode, dasc_stream_t stream) {
  if (!shape) return DASC_E_INVAL;
  size_t need = 0;
  const int rc = dasc_refresh_workspace_bytes(shape, n_req, W, &need);
  if (rc != DASC_OK) return rc;
  if (need > size_t(DASC_NOALLOC_SCRATCH_BYTES)) return DASC_E_SCRATCH;
  return dasc::refresh_impl(shape, layer, inv_row, states, n_pool, slot, k, v, g, beta, n_req, W,
                            init_mode, nullptr, 0, true, DASC_REFRESH_KERNEL_AUTO, stream);
}
