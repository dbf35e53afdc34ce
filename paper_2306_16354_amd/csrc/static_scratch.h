// The fixed scratch array of slhc_knn_graph_static (static_scratch.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace slhc {

// Holds the float16 copy and the buffers of the half-precision engine up to about 300 000 x 128; larger inputs go through the list
// kernels, which need one half norm per row only.
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)128 << 20;
// Its address on the current device.
hipError_t static_scratch_address(void** out);

}  // namespace slhc
