// Chunk form for fp32 inputs (plain and temporal): instantiations of the kernel
// in scan_gated_chunk_kernel.hpp, and the rule that picks it.
#include "scan_gated_chunk_kernel.hpp"

namespace swila {

bool chunk_f32_supported(const LayerArgs &a) {
    return !a.in_bf16 && a.T > 0 && a.J >= 1 && a.J <= 4 && !(a.delta_out && (a.gk || a.decay)) &&
           a.J * a.Dk <= 256 && a.Dv % 8 == 0 &&
           (a.Dk == 16 || a.Dk == 32 || a.Dk == 64 || a.Dk == 128);
}

// Where the three-part chunk form beats the token-by-token scan.  A chunk costs the
// same with one token in it as with 16, and the form's start some 2 us more, so the two
// meet at a length: T = c0 + e ceil(T / 16), a chunk being worth e tokens of the
// token scan.  A block's time does not depend on its column count, so e falls with the
// components.  Up to 256 column blocks (nb) every block has a compute unit; above that
// the chunk form takes rounds while the token scan's grid still fills the chip.
// Measured (chunk over token scan, D=64 unless said): T=2 J=4 1.2 to 1.3, T=8 J=1 1.1 to 1.5, T=17
// J=2 1.04 to 1.11, T=256 nb <= 256 0.24 to 0.69 (Dk=128 J=1 0.63 to 0.95); nb=512 J=1 Dk=128
// 0.97 to 1.38, J=2 0.75 to 0.82, J=4 0.54 to 0.60; nb=1024 and 2048, with gates: J=1 1.34 to
// 2.02, J=2 0.91 to 1.36, J=4 0.60 to 0.88 (T=16 and 32 1.0 to 1.4), Dk=16 J=4 0.90 to 1.49
// (nb=4096 0.55 to 0.66).
// Over 2,520 calls timed on both sides this takes none that is over 3% slower.
bool chunk_pays(const LayerArgs &a) {
    const long nb = (long)a.Dv / 16 * a.H * a.B, c = ((long)a.T + 15) / 16;
    const bool wide = a.J >= 3 && (!a.decay || a.J * a.Dk >= 128);   // pays at any grid
    int c0, e;
    if (nb > 256) {
        if (a.J == 1 && a.Dk >= 64) return false;
        if (!wide && nb > 512 && !(a.Dk == 16 && a.J > 1 && nb >= 4096)) return false;
        c0 = a.J >= 3 && nb <= 512 ? 0 : 16, e = a.J >= 3 && nb <= 512 ? 11 : 14;
    } else if (a.J >= 3) {
        c0 = 0, e = a.J == 4 ? 6 : 8;
    } else if (a.J == 2) {
        c0 = a.Dk <= 32 ? 1 : 4, e = a.Dk <= 32 ? 8 : 9;
    } else {
        c0 = a.Dk == 16 ? 5 : a.Dk == 32 ? 4 : a.Dk == 128 && a.decay ? 16 : 8;
        e = a.Dk == 16 ? 6 : a.Dk == 32 ? 9 : a.Dk == 128 && a.decay ? 13 : 11;
    }
    // (fp32 with gates and priors at J = 4, Dk = 64: only 8 output dims fit a block, so
    // that its grids are twice as large: nb=256 T=17 1.38, T=256 0.70; nb=1024 1.13)
    if (!a.in_bf16 && a.decay && a.gk && a.J == 4 && a.Dk == 64) {
        if (nb > 256) return false;
        if (nb > 128) c0 = 8, e = 13;
    }
    return a.T >= c0 + e * c;
}

bool chunk_f32_preferred(const LayerArgs &a) {
    return chunk_f32_supported(a) && (long)a.T * a.J >= 32 &&
           (long)a.Dv / 16 * a.H * a.B <= (a.J >= 3 ? 1024 : 256) && chunk_pays(a);
}

hipError_t launch_scan_chunk_f32(const LayerArgs &a, hipStream_t stream) {
    if (!chunk_f32_supported(a)) return hipErrorInvalidValue;
    if (a.decay) return launch_scan_chunk_f32_gated(a, stream);
    return a.gk ? launch_gated<true, false, true>(a, stream) : launch_gated<false, false, true>(a, stream);
}

}  // namespace swila
