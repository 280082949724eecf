// Kernel launchers that only note the stream they were given (fake_hip.h).
#include "fake_hip.h"
#include "kernels.h"

namespace merak {
static hipError_t on(hipStream_t s) {
  fake::launch(s);
  return hipSuccess;
}
hipError_t launch_gemm(int, bool, bool, int, const GemmProblem*, int, hipStream_t s, bool) { return on(s); }
hipError_t launch_layernorm_fwd(int, int, int, float, const void*, const void*, const void*, void*, float*, float*,
                                hipStream_t s, int, int) { return on(s); }
hipError_t launch_layernorm_bwd(int, int, int, const void*, const void*, const float*, const float*, const void*,
                                const void*, void*, hipStream_t s, int, int) { return on(s); }
hipError_t launch_layernorm_bwd_full(int, int, int, const void*, const void*, const float*, const float*, const void*,
                                     const void*, void*, float*, float*, int, float*, hipStream_t s) { return on(s); }
hipError_t launch_column_partials(int, int, int, const void*, float*, hipStream_t s) { return on(s); }
hipError_t launch_reduce_partials(int, int, const float*, float*, int, hipStream_t s) { return on(s); }
hipError_t launch_column_partials_batch(int, const ColPartialJob*, int, hipStream_t s) { return on(s); }
hipError_t launch_reduce_partials_batch(const ReduceJob*, int, hipStream_t s) { return on(s); }
hipError_t noalloc_scratch(float**) { return hipErrorNotSupported; }
hipError_t launch_count_nonfinite(int, const void*, long long, unsigned long long*, hipStream_t s) { return on(s); }
hipError_t launch_attention_fwd(int, int, int, int, int, const void*, void*, float*, hipStream_t s, int, int) {
  return on(s);
}
hipError_t launch_attention_bwd(int, int, int, int, int, const void*, const void*, const float*, const void*, void*,
                                float*, hipStream_t s, int, int) { return on(s); }
}  // namespace merak
