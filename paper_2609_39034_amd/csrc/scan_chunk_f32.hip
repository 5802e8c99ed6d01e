// Chunk form for fp32 inputs (plain and temporal): instantiations of the kernel
// in scan_gated_chunk_kernel.hpp, and the rule that picks it.
#include "scan_gated_chunk_kernel.hpp"

namespace swila {

bool chunk_f32_supported(const LayerArgs &a) {
    return !a.in_bf16 && a.T > 0 && a.J >= 1 && a.J <= 4 && !(a.delta_out && (a.gk || a.decay)) &&
           a.J * a.Dk <= 256 && a.Dv % 8 == 0 &&
           (a.Dk == 16 || a.Dk == 32 || a.Dk == 64 || a.Dk == 128);
}

// Where the chunk form beats the token-by-token scan.  A block's time does not
// depend on its column count, so its rate is that of a full block (J = 3 and 4:
// most of the 64 columns) only with enough components, while the token scan's grows
// until the chip is full: with nb = Dv / 16 * H * B, at T = 512 the chunk form is
// 1.2 to 4.6 times as fast for every J and Dk at nb <= 256 (D=64 J=4 B=4 H=16: 86
// against 249 us; D=128 J=1: 94 against 165, gated 139 against 166); at nb = 1024
// 1.04 to 2.2 times for J = 4 (D=64: 177 against 240 us, gated 234 against 393) but
// 0.6 to 1.0 for J = 1 and 2 at Dk >= 64; at nb = 4096 0.85 to 1.6 for J = 4.
// A chunk costs the same with one token in it as with 16, and the chunk form's start
// some 2 us more: the two meet at T = 2 for J = 4 (Dk = 64: 6.7 us), 10 to 12 for
// J = 2 (Dk = 16: 5.5 us) and 30 for J = 1 (Dk = 128: 12 us).
bool chunk_f32_preferred(const LayerArgs &a) {
    return chunk_f32_supported(a) && a.T * a.J >= 32 &&
           (long)a.Dv / 16 * a.H * a.B <= (a.J >= 3 ? 1024 : 256);
}

hipError_t launch_scan_chunk_f32(const LayerArgs &a, hipStream_t stream) {
    if (!chunk_f32_supported(a)) return hipErrorInvalidValue;
    if (a.decay) return launch_scan_chunk_f32_gated(a, stream);
    return a.gk ? launch_gated<true, false, true>(a, stream) : launch_gated<false, false, true>(a, stream);
}

}  // namespace swila
