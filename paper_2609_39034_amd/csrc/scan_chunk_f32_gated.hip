// Chunk form for fp32 inputs with gates: instantiations of the kernel in
// scan_gated_chunk_kernel.hpp.
#include "scan_gated_chunk_kernel.hpp"

namespace swila {

hipError_t launch_scan_chunk_f32_gated(const LayerArgs &a, hipStream_t stream) {
    if (!a.decay || !chunk_f32_supported(a)) return hipErrorInvalidValue;
    return a.gk ? launch_gated<true, true, true>(a, stream) : launch_gated<false, true, true>(a, stream);
}

}  // namespace swila
