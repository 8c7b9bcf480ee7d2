// The GEMM kernels of one mode: all-gather of column chunks.
#include <hip/hip_runtime.h>

#include <atomic>

#define PK_DEFINE_LAUNCH
#include "pk_tiles.h"

namespace pk {
template pk_status launch_gemm<EPI_AGK>(GemmArgs, int, bool, bool, bool, int, hipStream_t);
}
