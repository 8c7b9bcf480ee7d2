// The GEMM kernels of one mode: reduce-scatter, bf16 slots.
#include <hip/hip_runtime.h>

#include <atomic>

#define PK_DEFINE_LAUNCH
#include "pk_tiles.h"

namespace pk {
template pk_status launch_gemm<EPI_RS16>(GemmArgs, int, bool, bool, bool, int, hipStream_t);
}
