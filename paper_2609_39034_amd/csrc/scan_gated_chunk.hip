// Gated SwiLA (App. B.4) on the matrix cores, bf16 inputs: instantiations of the
// kernel in scan_gated_chunk_kernel.hpp.
#include "scan_gated_chunk_kernel.hpp"

namespace swila {

bool gated_chunk_supported(const LayerArgs &a) {
    // the temporal form: where the gate waves apply (J * Dk <= 256)
    return a.in_bf16 && a.decay && !a.delta_out && !a.ckpt && a.J >= 1 && a.J <= 4 &&
           a.J * a.Dk <= (a.gk ? 256 : 512) && a.Dv % 8 == 0 &&
           (a.Dk == 16 || a.Dk == 32 || a.Dk == 64 || a.Dk == 128);
}

hipError_t launch_scan_gated_chunk(const LayerArgs &a, hipStream_t stream) {
    if (!gated_chunk_supported(a) || a.T <= 0) return hipErrorInvalidValue;
    if (a.J * a.Dk > 384) return launch_scan_gated_chunk_wide(a, stream);   // both sides: that file
    return a.gk ? launch_gated<true, true, false>(a, stream) : launch_gated<false, true, false>(a, stream);
}

}  // namespace swila
