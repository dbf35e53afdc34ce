// The fixed scratch array of slhc_knn_graph_static, and nothing else: the runtime gives a GPU the code and the variables of
// a source file when something of that file is first used there, so a GPU holds this array from the first call of that entry
// point on and not because the library runs on it.
#include <hip/hip_runtime.h>
#include "static_scratch.h"

namespace slhc {

static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

hipError_t static_scratch_address(void** out) { return hipGetSymbolAddress(out, HIP_SYMBOL(scratch)); }

}  // namespace slhc
