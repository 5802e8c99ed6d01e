// Chunk form of Gated SwiLA on the matrix cores (App. B.4, eq. pre-decay with
// one gate per key dimension, eq. gate-elementwise tied across the output
// index): bf16 inputs, fp32 state.
//
// Per component j and output dim d the recurrence is
//   w~_t = a_t (.) w_{t-1},   delta_t = v_t - k_t . w~_t,   w_t = w~_t + c_t k_t,
// c_t = beta r delta (r from eq. responsibility at the decayed state), with
// a_t = sigmoid(decay logit) in (0,1)^Dk.  Inside a chunk of 16 tokens that
// starts from S, with L_t = sum_{u<=t} log a_u (per key index, from the chunk
// start) and E_t = e^{L_t}:
//   w~_t = E_t (.) S + sum_{s<t} (E_t / E_s) (.) k_s c_s
//   pred_t  = (k_t (.) E_t) . S + sum_{s<t} G_ts c_s,   G_ts = sum_i k_ti k_si e^{L_ti - L_si}
//   q_t.w_t = (q_t (.) E_t) . S + sum_{s<=t} QG_ts c_s, QG_ts = sum_i q_ti k_si e^{L_ti - L_si}
//   S'      = E_C (.) S + sum_s (k_s (.) E_C / E_s) c_s.
// G and QG are formed as (K (.) E)(K (.) E^-1)^T on the matrix cores while
// every E^-1 stays below e^{40}.  E^-1 is the running product of 1 + e^{-x}
// over the chunk's decay logits x (1 / sigmoid), one exponential per element,
// and E its reciprocal; a chunk whose gates decay further (some E^-1_C above
// e^{40}, or a gate closed altogether) keeps its gates a_t instead and takes every
// factor as the product of the gates between its two tokens
// (gated_chunk_common.hpp).  The scaled operands are fp32: each is split into a
// bf16 high part and a bf16 residual, and the hi*hi + hi*lo + lo*hi products
// are summed (about 2^-16 relative per product, fp32 accumulation).  With the
// temporal priors (App. B.3), a form that had only the token-by-token scan's fp32
// arithmetic before, each is split into three parts and six products are summed,
// which keeps all 24 bits, and E^-1 is formed in 64 bits: the state's error against fp64
// is 1.3e-7 to 1.5e-7 over lengths of 17 to 4096, that of o 1.1e-7 (token scan 1.4e-7
// to 1.5e-7, 1.2e-7).  A
// component's gates differ from the others', so each component has its own
// Gram matrices and scaled operands: tile wave j holds the state columns of
// component j.
//
// Block = one head (b, h) and DB output dims with all J components (J <= 4,
// J * Dk <= 384): J tile waves (wave j: the Dk x DB state tile of component j
// in accumulator registers), one sequential wave (one lane per column), three
// helper waves and, up to J * Dk = 256, one or two gate waves.  Per
// chunk n, between two block barriers:
//   phase A  sequential wave: the chunk's 16-token recurrence -> C_n
//            tile waves: retrieval of chunk n-1 (needs C_{n-1}); Q_n S_n and
//              the update operand of chunk n; K_{n+1} (.) E_{n+1}, Q_{n+1} (.)
//              E_{n+1}, G_{n+1} for the next recurrence and QG_{n+1}
//            gate waves: E^-1 of chunk n+2 (without them the tile waves, of
//              chunk n+1, each its component's)
//            helper waves: pi^q_n, the output of chunk n-2, and the inputs of
//              chunk n+2 but its decay logits (HBM -> registers -> LDS)
//   phase B  tile waves: S_{n+1} = E_C (.) S_n + U_n^T C_n and
//              P_{n+1} = (K_{n+1} (.) E_{n+1}) S_{n+1} for the next recurrence;
//            sequential wave: beta, key-prior logits and v of chunk n+1;
//            helper waves: the decay logits of chunk n+2 (no gate waves), the loads
//              of n+3; temporal: the running query prior over chunk n, g^k pi^k of
//              chunk n+2.
//
// Bound: the tile waves' operands (phase A 3,500 cycles a chunk at Dk = 64, the
// sequential wave 2,900 on the SIMD it shares with one of them), then phase B's
// 1,050.  One launch at B=4 H=8 T=2048 D=64 J=4, before (deferred updates as
// multiply-adds, gates by the tile waves) and now: 0.364 -> 0.287 ms; with the
// temporal priors, before on the token-by-token scan: 1.261 -> 0.404 ms.
//
// The same kernel evaluates fp32 inputs (F32), with or without gates (GT) and
// temporal priors: K and Q are then fp32 operands like the state, every operand
// is split into three parts, and without gates E = 1.
//
// This header holds the kernel template and its launch dispatch; bf16 inputs,
// fp32 inputs and fp32 inputs with gates are instantiated in translation units of
// their own (scan_gated_chunk.hip, scan_chunk_f32.hip, scan_chunk_f32_gated.hip).
#pragma once
#include <type_traits>

#include "gated_chunk_common.hpp"
#include "launch.hpp"

namespace swila {
namespace {

constexpr int kGH = 3;               // helper waves
// Roles of a block's waves, four bits each from wave 0 up (0: wave x has role x).
// Wave x runs on SIMD x mod 4, and its older waves go first.  With nine or ten
// waves some SIMDs have three: the sequential wave takes one that has two and no
// gate wave, and the gate waves go before the helpers; with six or seven it has one
// to itself.  Against roles in order, B=4 H=8 T=512 Dv=64: four tile and one gate wave
// (Dk=32, bf16 gated) 75.9 -> 61.9 us, three and two (Dk=64) 70.7 -> 67.5, two and one
// (Dk=32) 60.3 -> 53.4.  Eight waves stay in order (J = 3 with one gate wave and J = 2
// with two: the other orders tried were 3 to 12% slower).
template <int J, int NG>
constexpr uint64_t wave_roles() {
    return J == 4 && NG == 2 ? 0x6784593210ull   // tiles, gate, helper, sequential, gate, helpers
           : J == 4 && NG == 1 ? 0x765483210ull  // tiles, gate, sequential, helpers
           : J == 3 && NG == 2 ? 0x654873210ull  // tiles, sequential, gates, helpers
           : J == 2 && NG == 1 ? 0x5432610ull    // tiles, gate, sequential, helpers
           : J == 1 && NG == 1 ? 0x432150ull     // tile, gate, sequential, helpers
                               : 0;
}
// input y of a 16-byte piece (y a compile-time index)
template <bool F32>
__device__ __forceinline__ float piece(const uint4 &r, int y) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
    return F32 ? __uint_as_float(w[y % 4])
               : __uint_as_float(y % 2 ? w[y / 2 % 4] & 0xffff0000u : w[y / 2 % 4] << 16);
}

// TP: with the temporal priors (App. B.3); GT: with gates; F32: fp32 inputs.
template <int DK, int J, int DB, bool TP, bool GT, bool F32>
struct GCfg {
    using In = typename std::conditional<F32, float, uint16_t>::type;
    static constexpr int E = F32 ? 4 : 8;    // input elements per 16 bytes
    static constexpr int IT = DK / 16;       // 16-row key tiles
    static constexpr int N = J * DB;         // columns, col = j * DB + dd
    static constexpr int JP = J == 3 ? 4 : J;
    // Where three chunks of E^-1 fit the LDS, gate waves of their own form them two
    // chunks ahead (two key indices a lane, straight from HBM); else the tile waves
    // do, from the decay logits in LDS.
    static constexpr bool HG = GT && J * DK <= 256;
    static constexpr int NG = HG ? ceil_div_c(J * DK / 2, 64) : 0;   // gate waves
    static constexpr int NWAVE = J + 1 + kGH + NG;
    static constexpr int NEI = HG ? 3 : GT ? 1 : 0;   // slots of E^-1; E_C
    static constexpr int NEC = HG ? 3 : GT ? 2 : 0;
    static constexpr int SD = 16 / JP;       // output dims per 16 sequential lanes
    // The scaled units of the sequential wave, and back.  The temporal form and
    // fp32 inputs take none: each conversion is one more rounding of v, the
    // predictions and the coefficients, and a rounding of d grows by d^2 in the
    // exponential.
    static constexpr bool SCALED = !TP && !F32;
    static constexpr float S = SCALED ? kS : 1.0f, IS = SCALED ? kInvS : 1.0f;
    static constexpr int KP = DK + 4;        // bf16 row pitch of the K, Q tiles
    static constexpr int LP = DK + 4;        // fp32 row pitch of E^-1 (or the gates)
    static constexpr int CP = kGC + 4;       // [column][token] row pitch
    static constexpr int NP = N + 4;         // [token][column] row pitch
    static_assert(J >= 1 && J <= 4 && J * DK <= (F32 || TP ? 256 : 384), "LDS budget of the gated chunk form");
    static_assert(GT || F32, "bf16 inputs without gates run the plain chunk scan");
    static_assert(DB == 8 || DB == 16, "column block");
    static_assert(DB * JP <= 64, "one sequential wave");
};

template <int DK, int J, int DB, bool TP, bool GT, bool F32>
struct GSmem {
    using C = GCfg<DK, J, DB, TP, GT, F32>;
    using In = typename C::In;
    // chunk inputs, chunk m in slot m % 3
    alignas(16) In k[3][kGC][C::KP];
    alignas(16) In q[3][kGC][C::KP];
    alignas(16) In lq[3][kGC][C::N];   // [token][j * DB + dd]
    // decay logits of the next chunk to take its gates (tile waves' gates)
    alignas(16) uint16_t g[C::HG || !GT ? 1 : kGC][C::HG || !GT ? 8 : J * DK];
    // E^-1 of chunk m (its gates a_t in a deep chunk), and E_C, in
    // slots m % NEI and m % NEC; with gate waves, whether the chunk is deep
    alignas(16) float ei[GT ? C::NEI : 1][GT ? J : 1][GT ? kGC : 1][GT ? C::LP : 4];
    alignas(16) float ec[GT ? C::NEC : 1][GT ? J : 1][GT ? DK : 4];
    int deep[3][J];
    // for the sequential wave, chunk m in m & 1: {beta, key-prior logit (times log2(e)
    // in scaled units)} [column][token] (beta = 0 past the end) and s v [dim][token]; temporal: {beta,
    // g^k pi^k} and 1 - g^k [dim][token]
    alignas(16) float2 sq[2][C::N][kGC + 2];
    // (J = 3: row DB zeros, the padding lanes')
    alignas(16) float vs[2][DB + (J == 3)][kGC + 4];
    alignas(16) float gs[TP ? 2 : 1][TP ? DB : 1][kGC + 4];
    alignas(16) In lk[TP ? 2 : 1][TP ? kGC : 1][TP ? C::N : 8];   // temporal: key-prior logits
    float gq[TP ? 3 : 1][TP ? kGC : 1][TP ? DB : 1];        // temporal: g^q, chunk m in m % 3
    // -G of chunk m in m & 1, as A operands of the sequential wave's 4x4 products:
    // [j][s][i][m] = the value of token 4 m + i (later than s); and its first
    // subdiagonal, [j][s] = that of token s + 1
    alignas(16) float gt[2][J][kGC][kGC];
    alignas(16) float gsub[2][J][kGC];
    // chunk-start predictions, times s [column][token] (J = 3: row N zeros, the padding
    // lanes')
    alignas(16) float p[C::N + (J == 3)][C::CP];
    // coefficients [column][token], chunk m in m & 1 (row N: the idle lanes')
    alignas(16) float c[2][C::N + 1][C::CP];
    float pq[2][kGC][C::NP];                 // pi^q [token][column]
    float py[2][kGC][C::NP];                 // pi^q * retrieval [token][column]
};

// Each role runs its whole chunk loop in a branch of its own, so that the
// registers one role keeps across chunks are not held by the others; every
// role meets the same block barriers in the same order: four in the prologue,
// two per chunk (e(n): C_n and chunk n + 2 published; i(n+1): P_{n+1}
// published), one in the epilogue.
// (Nine and ten waves a block cap a lane at 168 registers.  Four instantiations spill,
// 8 to 12 bytes a lane: gates and priors, bf16 <32, 4, 8>, <64, 4, 16> and
// <128, 1, 16>, fp32 <32, 4, 16>.)
template <int DK, int J, int DB, bool TP, bool GT, bool F32>
__global__ __launch_bounds__((64 * GCfg<DK, J, DB, TP, GT, F32>::NWAVE)) void scan_gated_chunk_kernel(LayerArgs a) {
    using C = GCfg<DK, J, DB, TP, GT, F32>;
    using In = typename C::In;
    constexpr int IT = C::IT, N = C::N, JP = C::JP;
    constexpr bool HG = C::HG;
    // the form that can serve as the backward's recompute (delta_out, ckpt, no o)
    constexpr bool AX = F32 && !GT && !TP;
    // the temporal form and fp32 inputs keep the precision of the token-by-token
    // scan, on which they ran before: three parts
    constexpr int NP = TP || F32 ? 3 : 2;
    __shared__ GSmem<DK, J, DB, TP, GT, F32> sm;

    const int tid = threadIdx.x;
    // role w of this wave: 0 .. J-1 tile, J sequential, then the helpers, then the
    // gate waves
    const int wx = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
    constexpr uint64_t kRoles = wave_roles<J, C::NG>();
    const int w = kRoles ? (int)((kRoles >> (4 * wx)) & 15) : wx;
    const int tl = lane % 16, lg = lane / 16;
    const int H = a.H, T = a.T, Dv = a.Dv;
    int db, hh;
    gated_coords(blockIdx.x, Dv / DB, a.B * H, db, hh);
    const int d0 = db * DB, h = hh % H, b = hh / H;
    const int NCH = (T + kGC - 1) / kGC;

    if (w < J) {
        // ================= tile wave j: the state of component j =================
        // state S^j rows 16 it + 4 lg + r, column tl (a real column when tl < DB)
        const int tj = w;
        const bool tvalid = tl < DB;
        const int tcol = tj * DB + (tvalid ? tl : 0);
        // E^-1 (in a deep chunk the gates) of chunk m, [token][key index]
        auto ei_of = [&](int m) { return sm.ei[HG ? m % 3 : 0][GT ? tj : 0]; };
        floatx4 W[IT];
        S4<NP> Kp[IT];   // K_m (.) E_m for the next chunk m, A operand (rows t = tl)
        S4<NP> Qe[IT];   // Q_m (.) E_m for the next chunk m (rows t = tl)
        S4<NP> U[IT];    // update operand of chunk n: rows i = 16 it + tl, columns s = 4 lg + m
        // Q S and tril(QG) (A operand) of the chunk whose retrieval is pending
        // (r), and of the chunk after it (q)
        floatx4 Y0r = floatx4{0.f, 0.f, 0.f, 0.f}, Y0q = floatx4{0.f, 0.f, 0.f, 0.f};
        S4<NP> QGr = zero4<NP>(), QGq = zero4<NP>();
        bool deep_n = false, deep_n1 = false;   // chunk n, n+1 past the factorised Gram products

        // E^-1 (in a deep chunk the gates) and E_C of chunk m for component tj from
        // its decay logits (lane: key indices 2 lane and 2 lane + 1); returns whether the
        // chunk is deep.
        auto log_gates = [&](int m) {
            if constexpr (!GT) {
                return false;
            } else if constexpr (HG) {   // formed by the gate waves
                return sm.deep[m % 3][tj] != 0;
            } else {
            static_assert(HG || !GT || DK == 128, "tile waves form the gates of J = 3, Dk = 128 alone");
            const int nt = min(kGC, T - m * kGC);
            bool deep = false;
            auto *const EI = ei_of(m);
            // two adjacent key indices per lane
            const int i = 2 * lane;
            uint32_t x[kGC];
#pragma unroll
            for (int t = 0; t < kGC; ++t)
                x[t] = *reinterpret_cast<const uint32_t *>(&sm.g[t][tj * DK + i]);
            float c0 = 1.0f, c1 = 1.0f;
#pragma unroll
            for (int t = 0; t < kGC; ++t) {
                const float f0 = 1.0f + __builtin_amdgcn_exp2f(-kLog2e * __uint_as_float(x[t] << 16));
                const float f1 =
                    1.0f + __builtin_amdgcn_exp2f(-kLog2e * __uint_as_float(x[t] & 0xffff0000u));
                c0 *= t < nt ? f0 : 1.0f;
                c1 *= t < nt ? f1 : 1.0f;
                *reinterpret_cast<float2 *>(&EI[t][i]) = make_float2(c0, c1);
            }
            *reinterpret_cast<float2 *>(&sm.ec[m % C::NEC][tj][i]) = make_float2(rcp_fast(c0), rcp_fast(c1));
            deep = !(c0 <= kGramEinv) || !(c1 <= kGramEinv);
            if (__any(deep) == 0) return false;
            // deep chunk: the gates, in place of E^-1
            float l0 = 1.0f, l1 = 1.0f;
#pragma unroll
            for (int t = 0; t < kGC; ++t) {
                const float a0 = t < nt ? sigmoid(__uint_as_float(x[t] << 16)) : 1.0f;
                const float a1 = t < nt ? sigmoid(__uint_as_float(x[t] & 0xffff0000u)) : 1.0f;
                l0 *= a0, l1 *= a1;
                *reinterpret_cast<float2 *>(&EI[t][i]) = make_float2(a0, a1);
            }
            *reinterpret_cast<float2 *>(&sm.ec[m % C::NEC][tj][i]) = make_float2(l0, l1);
            return true;
            }
        };

        // four inputs of row tl of X, key indices 16 it + 4 lg .. + 3, times f
        auto row4 = [&](const In (*X)[C::KP], int it, float4 f) {
            const float4 x = in4(&X[tl][16 * it + 4 * lg]);
            return GT ? split4<NP>(x.x * f.x, x.y * f.y, x.z * f.z, x.w * f.w)
                      : split4<NP>(x.x, x.y, x.z, x.w);
        };
        // the operands of chunk m: Kp, Qe, G_m (for the sequential wave) and QG_m
        auto gram = [&](int m, bool pair) {
            const int s3 = m % 3;
            auto *const EI = ei_of(m);
            floatx4 g = floatx4{0.f, 0.f, 0.f, 0.f}, qg = floatx4{0.f, 0.f, 0.f, 0.f};
            if (!pair) {
                // E^-1 and E at rows tl, key indices 16 it + 4 lg .. + 3; K (.) E^-1
                // at rows s = tl
                auto operands = [&](int it) {
                    if constexpr (GT) {
                        const float4 x = *reinterpret_cast<const float4 *>(&EI[tl][16 * it + 4 * lg]);
                        const float4 er = make_float4(rcp_fast(x.x), rcp_fast(x.y), rcp_fast(x.z), rcp_fast(x.w));
                        Kp[it] = row4(sm.k[s3], it, er);
                        Qe[it] = row4(sm.q[s3], it, er);
                        return row4(sm.k[s3], it, x);
                    } else {
                        Kp[it] = row4(sm.k[s3], it, float4{});
                        Qe[it] = row4(sm.q[s3], it, float4{});
                        return Kp[it];
                    }
                };
                if constexpr (IT == 1) {
                    const S4<NP> kinv = operands(0);
                    g = mm<NP>(Kp[0], kinv, g);      // D[t = 4 lg + r][s = tl] = G_ts
                    qg = mm<NP>(kinv, Qe[0], qg);    // D[s = 4 lg + r][t = tl] = QG_ts
                } else {
#pragma unroll
                    for (int it = 0; it < IT; it += 2) {
                        const S4<NP> k0 = operands(it), k1 = operands(it + 1);
                        g = mmx2<NP>(Kp[it], Kp[it + 1], k0, k1, g);
                        qg = mmx2<NP>(k0, k1, Qe[it], Qe[it + 1], qg);
                    }
                }
                // lane (tl, lg) holds QG[t = tl][s = 4 lg + r]: the A operand of the retrieval
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (4 * lg + r > tl) qg[r] = 0.0f;
            } else if constexpr (GT) {
                deep_grams<DK, NP>(EI, sm.k[s3], sm.q[s3], tl, lg, g, qg);
#pragma unroll
                for (int it = 0; it < IT; ++it) {
                    const float4 er = decay_to(EI, tl, 16 * it + 4 * lg);
                    Kp[it] = row4(sm.k[s3], it, er);
                    Qe[it] = row4(sm.q[s3], it, er);
                }
            }
            // lane (tl, lg) holds G of tokens 4 lg + r, column s = tl
#pragma unroll
            for (int r = 0; r < 4; ++r) sm.gt[m & 1][tj][tl][4 * r + lg] = -g[r];
            const int nx = tl + 1;
            const float lo = nx & 1 ? g[1] : g[0], hi = nx & 1 ? g[3] : g[2];
            if (nx >> 2 == lg) sm.gsub[m & 1][tj][tl] = -(nx & 2 ? hi : lo);
            QGq = split4<NP>(qg);
        };
        // for the next chunk, from its start state S: the predictions P = Kp S
        // for the sequential wave, in its units, and Q S (Y0q)
        auto predict = [&]() {
            floatx4 pacc = floatx4{0.f, 0.f, 0.f, 0.f}, y0 = floatx4{0.f, 0.f, 0.f, 0.f};
            if constexpr (IT == 1) {
                const S4<NP> ws = split4<NP>(W[0]);
                pacc = mm<NP>(Kp[0], ws, pacc);   // D[t][col]
                y0 = mm<NP>(Qe[0], ws, y0);
            } else {
#pragma unroll
                for (int it = 0; it < IT; it += 2) {
                    const S4<NP> w0 = split4<NP>(W[it]), w1 = split4<NP>(W[it + 1]);
                    pacc = mmx2<NP>(Kp[it], Kp[it + 1], w0, w1, pacc);
                    y0 = mmx2<NP>(Qe[it], Qe[it + 1], w0, w1, y0);
                }
            }
            if (tvalid)
                *reinterpret_cast<float4 *>(&sm.p[tcol][4 * lg]) =
                    make_float4(C::S * pacc[0], C::S * pacc[1], C::S * pacc[2], C::S * pacc[3]);
            Y0q = y0;
        };
        // C of chunk m as the B operand: rows s = 4 lg .. + 3, column tl
        auto coeffs = [&](int m) {
            const float4 c4 = *reinterpret_cast<const float4 *>(&sm.c[m & 1][tcol][4 * lg]);
            return tvalid ? split4<NP>(c4.x, c4.y, c4.z, c4.w) : zero4<NP>();
        };
        // retrieval of chunk m: Y = Y0 + tril(QG) C, times pi^q, to py
        auto retrieve = [&](int m) {
            float4 c4 = *reinterpret_cast<const float4 *>(&sm.c[m & 1][tcol][4 * lg]);
            if (!tvalid) c4 = make_float4(0.f, 0.f, 0.f, 0.f);
            // A coefficient that is not finite (an input that is not) would reach the
            // tokens before its own too, as 0 times it: such ones are taken out of the
            // product, and the column's tokens from the first on set to NaN.  (The gated
            // form on bf16 inputs leaves that out, as the plain chunk scan does.)
            const bool odd = NP == 3 && __builtin_amdgcn_ballot_w64(!(fabsf((c4.x + c4.y) + (c4.z + c4.w)) < INFINITY)) != 0;
            int first = kGC;
            if (odd) {
                float *const c = &c4.x;
#pragma unroll
                for (int r = 3; r >= 0; --r)
                    if (!(fabsf(c[r]) < INFINITY)) c[r] = 0.f, first = 4 * lg + r;
                first = min(first, __shfl_xor(first, 16));
                first = min(first, __shfl_xor(first, 32));
            }
            floatx4 y = mm<NP>(QGr, split4<NP>(c4.x, c4.y, c4.z, c4.w), Y0r);   // D[t = 4 lg + r][col]
            if (odd) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (4 * lg + r >= first) y[r] = NAN;
            }
            if (tvalid) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int t = 4 * lg + r;
                    sm.py[m & 1][t][tcol] = sm.pq[m & 1][t][tcol] * y[r];
                }
            }
        };
        // what chunk n needs besides C_n: its Q S and tril(QG) for the retrieval
        // (from Y0q and QGq) and U_n (EI holds chunk n's E^-1 or gates)
        auto prepare = [&](int n, bool pair) {
            const int s3 = n % 3;
            auto *const EI = ei_of(n);
            Y0r = Y0q;
            QGr = QGq;
            // U[i][s] = K[s][i] E_C,i / E_s,i, i = 16 it + tl, s = 4 lg + m
            if (!pair) {
#pragma unroll
                for (int it = 0; it < IT; ++it) {
                    const int i = 16 * it + tl;
                    const float ecv = GT ? sm.ec[GT ? n % (GT ? C::NEC : 1) : 0][GT ? tj : 0][GT ? i : 0] : 1.0f;
                    float u[4];
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const int s = 4 * lg + m;
                        u[m] = GT ? bf(sm.k[s3][s][i]) * (ecv * EI[s][i]) : bf(sm.k[s3][s][i]);
                    }
                    U[it] = split4<NP>(u[0], u[1], u[2], u[3]);
                }
            } else if constexpr (GT) {
#pragma unroll
                for (int it = 0; it < IT; ++it) {
                    const int i = 16 * it + tl;
                    float u[4], f[4];
                    decay_after(EI, lg, i, f);
#pragma unroll
                    for (int m = 0; m < 4; ++m) u[m] = bf(sm.k[s3][4 * lg + m][i]) * f[m];
                    U[it] = split4<NP>(u[0], u[1], u[2], u[3]);
                }
            }
        };

#pragma unroll
        for (int it = 0; it < IT; ++it)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                W[it][r] = tvalid && a.state_in
                               ? a.state_in[(((size_t)b * H + h) * J + tj) * DK * Dv +
                                            (size_t)(16 * it + 4 * lg + r) * Dv + d0 + tl]
                               : 0.0f;
        block_sync_lds();   // prologue 1
        block_sync_lds();   // prologue 2: chunks 0 and 1 in LDS (the decay logits of 0)
        deep_n = log_gates(0);
        gram(0, deep_n);
        predict();          // P_0, Q_0 S_0
        block_sync_lds();   // prologue 3: the decay logits of chunk 0 read
        block_sync_lds();   // prologue 4: those of chunk 1 in LDS
        for (int n = 0; n < NCH; ++n) {
            // ---- phase A: everything that does not need C_n
            if constexpr (AX) {
                // the state before every kBwdChunk-th token, [b, h, interval, d, j, i]
                static_assert(kBwdChunk == 2 * kGC, "checkpoints every second chunk");
                if (a.ckpt && (n & 1) == 0 && tvalid) {
                    const int NC2 = (T + 2 * kGC - 1) / (2 * kGC);
                    float *dst = a.ckpt + (((((size_t)b * H + h) * NC2 + n / 2) * Dv + d0 + tl) * J + tj) * DK;
#pragma unroll
                    for (int it = 0; it < IT; ++it)
                        *reinterpret_cast<float4 *>(dst + 16 * it + 4 * lg) =
                            make_float4(W[it][0], W[it][1], W[it][2], W[it][3]);
                }
            }
            if (n >= 1) retrieve(n - 1);
            prepare(n, deep_n);
            if (n + 1 < NCH) {
                deep_n1 = log_gates(n + 1);
                gram(n + 1, deep_n1);
            }
            block_sync_lds();   // e(n)
            // ---- phase B: S_{n+1} = E_C (.) S_n + U_n^T C_n, then P_{n+1}, Q_{n+1} S_{n+1}
            const S4<NP> cb = coeffs(n);
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                if constexpr (GT) {
                    const float4 e4 = *reinterpret_cast<const float4 *>(&sm.ec[n % C::NEC][tj][16 * it + 4 * lg]);
                    W[it][0] *= e4.x;
                    W[it][1] *= e4.y;
                    W[it][2] *= e4.z;
                    W[it][3] *= e4.w;
                }
                W[it] = mm<NP>(U[it], cb, W[it]);
            }
            if (n + 1 < NCH) predict();
            deep_n = deep_n1;
            block_sync_lds();   // i(n+1)
        }
        retrieve(NCH - 1);
        block_sync_lds();   // epilogue
        if (tvalid && a.state_out) {
#pragma unroll
            for (int it = 0; it < IT; ++it)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    a.state_out[(((size_t)b * H + h) * J + tj) * DK * Dv +
                                (size_t)(16 * it + 4 * lg + r) * Dv + d0 + tl] = W[it][r];
        }
    } else if (w == J) {
        // ================= sequential wave: one lane per column =================
        // lane 16 x + SD j + y: component j of output dim SD x + y, so that four
        // adjacent lanes share a component (one block of the 4x4 products) and the
        // components of a dim lie in one row of 16 lanes
        const int sdd = lane / 16 * C::SD + lane % C::SD, sj = lane % 16 / C::SD;
        const bool sact = sdd < DB && sj < J;
        const int scol = sact ? sj * DB + sdd : 0, gj = sact ? sj : 0;
        const int scst = sact ? scol : N;
        // The padding component of J = 3 is summed with the others of its dim: its lanes
        // read rows of zeros, since another column's v or predictions would carry what is
        // not finite there to this dim.  (Lanes of no dim read column 0.)
        constexpr bool PAD = J == 3;
        const int spre = sact ? scol : PAD ? N : 0;
        const bool wres = a.resp && sact;
        auto lane_sum = [](float x) {
            if constexpr (JP >= 4) x += dpp_mov<0x124>(x);   // row_ror 4
            if constexpr (JP >= 2) x += dpp_mov<0x128>(x);   // row_ror 8
            return x;
        };
        auto lane_max = [](float x) {
            if constexpr (JP >= 4) x = fmaxf(x, dpp_mov<0x124>(x));
            if constexpr (JP >= 2) x = fmaxf(x, dpp_mov<0x128>(x));
            return x;
        };
        float sbeta[kGC], slk[kGC], sgs[TP ? kGC : 1];
        floatx4 sv[kGC / 4];
        const int vdd = sact ? sdd : PAD ? DB : 0;
        if constexpr (PAD)   // (read by this wave alone)
            if (lane < kGC) sm.p[N][lane] = sm.vs[0][DB][lane] = sm.vs[1][DB][lane] = 0.0f;
        // r_{t-1} of this lane's column (temporal), and that of the last token
        float rprev = 0.0f, rlast = 0.0f;
        if constexpr (TP) {
            if (sact)
                rprev = a.prior_in ? a.prior_in[(((size_t)b * H + h) * 2 * J + sj) * Dv + d0 + sdd]
                                   : 1.0f / J;
        }
        // beta, key-prior logits and v of chunk m
        auto seq_inputs = [&](int m) {
#pragma unroll
            for (int t2 = 0; t2 < kGC; t2 += 2) {
                const float4 x = *reinterpret_cast<const float4 *>(&sm.sq[m & 1][scol][t2]);
                // idle lanes (and the padding component of J = 3) carry no mass
                constexpr float none = TP ? 0.0f : -INFINITY;
                sbeta[t2] = sact ? x.x : 0.0f, slk[t2] = sact ? x.y : none;
                sbeta[t2 + 1] = sact ? x.z : 0.0f, slk[t2 + 1] = sact ? x.w : none;
            }
#pragma unroll
            for (int t4 = 0; t4 < kGC; t4 += 4) {
                const float4 x = *reinterpret_cast<const float4 *>(&sm.vs[m & 1][vdd][t4]);
                sv[t4 / 4] = floatx4{x.x, x.y, x.z, x.w};
                if constexpr (TP) {
                    const float4 y = *reinterpret_cast<const float4 *>(&sm.gs[m & 1][sact ? sdd : 0][t4]);
                    sgs[t4] = sact ? y.x : 0.f, sgs[t4 + 1] = sact ? y.y : 0.f;
                    sgs[t4 + 2] = sact ? y.z : 0.f, sgs[t4 + 3] = sact ? y.w : 0.f;
                }
            }
        };
        __builtin_amdgcn_s_setprio(3);   // (before its SIMD's tile wave)
        block_sync_lds();   // prologue 1
        block_sync_lds();   // prologue 2
        block_sync_lds();   // prologue 3
        seq_inputs(0);
        block_sync_lds();   // prologue 4
        for (int n = 0; n < NCH; ++n) {
            const int t0 = n * kGC, nt = min(kGC, T - t0), gs = n & 1;
            // ---- the token recurrence of chunk n, in scaled units.  The softmax
            // over j runs without subtracting its maximum: for logits and errors
            // of ordinary size its sum z stays far inside the fp32 range.  Should
            // z of some column and token leave [2^-100, 2^100], the chunk is run
            // again with the maximum subtracted (the bound of the plain chunk scan).
            // As there, the wave is bound by its instruction count: D holds v - pred
            // of the chunk's tokens, four to a register group, and a coefficient
            // reaches the next token by one multiply-add and the others as 4x4x1
            // products (a block's A operand is its component's -G), one batch a token.
            // In the forms that keep all 24 bits D holds -pred and v joins at the
            // token (one addition more): its 15 updates are rounded at the size of the
            // prediction and not of v, which was the whole excess of these forms'
            // error over the token scan's (2-norm of the state against
            // 64 bits at B=4 H=8 T=256 D=64 J=4, with E^-1 rounded once as well: bf16
            // gated temporal 2.8e-7 -> 1.5e-7, token scan 1.5e-7; fp32 gated 2.3e-7 ->
            // 1.2e-7, 1.4e-7; fp32 plain 2.3e-7 -> 1.7e-7, 3.2e-7).
            floatx4 D[kGC / 4], A[kGC];
            float cb[4], gsub[kGC];
            auto start = [&]() {
#pragma unroll
                for (int i = 0; i < kGC / 4; ++i) {
                    const float4 p4 = *reinterpret_cast<const float4 *>(&sm.p[spre][4 * i]);
                    const floatx4 p = floatx4{p4.x, p4.y, p4.z, p4.w};
                    D[i] = C::SCALED ? sv[i] - p : -p;
                }
            };
            // v - pred of token t, given what D collects
            auto error = [&](auto tag, float x) {
                constexpr int t = decltype(tag)::value;
                return C::SCALED ? x : sv[t / 4][t % 4] + x;
            };
            start();
#pragma unroll
            for (int i = 0; i < kGC; i += 4) {
                const float4 x = *reinterpret_cast<const float4 *>(&sm.gsub[gs][gj][i]);
                gsub[i] = x.x, gsub[i + 1] = x.y, gsub[i + 2] = x.z, gsub[i + 3] = x.w;
            }
            auto load_a = [&](int t) {   // the A operands of the updates by token t
                const float4 x = *reinterpret_cast<const float4 *>(&sm.gt[gs][gj][t][4 * (lane & 3)]);
                A[t] = floatx4{x.x, x.y, x.z, x.w};
            };
            load_a(0);
            load_a(1);
            // the later tokens of the chunk by the coefficient of token S (token
            // S + 1 has it), the group that is read next first
            auto defer = [&](auto tag, float cs) {
                constexpr int S = decltype(tag)::value;
#pragma unroll
                for (int m = (S + 2) / 4; m < kGC / 4; ++m)
                    D[m] = __builtin_amdgcn_mfma_f32_4x4x1f32(A[S][m], cs, D[m], 0, 0, 0);
            };
            const float rprev0 = rprev;
            float chk = 0.f, cprev = 0.f, d = error(ITag<0>{}, D[0][0]);
            auto keep_r = [&](int t, float rt, float dt) {
                if constexpr (AX) {   // the backward's recompute: delta of every token
                    if (sact && t < nt && a.delta_out)
                        a.delta_out[((((size_t)b * T + t0 + t) * H + h) * J + sj) * Dv + d0 + sdd] = C::IS * dt;
                }
                if (wres) {   // (tokens past the end stay in registers)
                    if (t < nt)
                        a.resp[((((size_t)b * T + t0 + t) * H + h) * J + sj) * Dv + d0 + sdd] = rt;
                }
                if constexpr (TP) {
                    rprev = rt;
                    rlast = t < nt ? rt : rlast;
                }
            };
            auto token = [&](auto tag) {
                constexpr int t = decltype(tag)::value;
                float ex;
                if constexpr (TP)   // key prior (1 - g^k) r_{t-1} + g^k pi^k
                    ex = __builtin_amdgcn_exp2f(-kS2 * d * d);
                else   // (log2(e) here: an fp32 logit times it may overflow, see slow)
                    ex = __builtin_amdgcn_exp2f(fmaf(C::SCALED ? -d : -kS2 * d, d, C::SCALED ? slk[t] : kLog2e * slk[t]));
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (t >= 1) defer(ITag<(t > 0 ? t - 1 : 0)>{}, cprev);
                __builtin_amdgcn_sched_barrier(0);
                const float bd = sbeta[t] * d;
                if constexpr (TP) ex *= fmaf(sgs[t], rprev, slk[t]);
                if constexpr (t + 2 < kGC - 2) load_a(t + 2);
                __builtin_amdgcn_sched_barrier(0);
                float z = ex;
                if constexpr (JP >= 4) z += dpp_mov<0x124>(z);   // row_ror 4
                const float bdex = bd * ex;
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (JP >= 2) z += dpp_mov<0x128>(z);   // row_ror 8
                const float iz = rcp_fast(z);
                // (one component: r = 1 whatever the exponent; not finite stays so)
                const float rt = J == 1 ? fmaf(0.0f, slk[t], 1.0f) : ex * iz;
                const float cs = J == 1 || TP ? bd * rt : bdex * iz;   // s c
                float dn = 0.f;
                if constexpr (t + 1 < kGC)
                    dn = error(ITag<(t + 1 < kGC ? t + 1 : 0)>{}, fmaf(gsub[t], cs, D[(t + 1) / 4][(t + 1) % 4]));
                cb[t & 3] = C::IS * cs;
                if ((t & 3) == 3)
                    *reinterpret_cast<float4 *>(&sm.c[gs][scst][t - 3]) =
                        make_float4(cb[0], cb[1], cb[2], cb[3]);
                keep_r(t, rt, d);
                if constexpr (J > 1) {
                    chk = fmaxf(fmaxf(z, iz), chk);
                    asm volatile("" : "+v"(chk));
                }
                cprev = cs;
                d = dn;
            };
            token(ITag<0>{}), token(ITag<1>{}), token(ITag<2>{}), token(ITag<3>{});
            token(ITag<4>{}), token(ITag<5>{}), token(ITag<6>{}), token(ITag<7>{});
            token(ITag<8>{}), token(ITag<9>{}), token(ITag<10>{}), token(ITag<11>{});
            token(ITag<12>{}), token(ITag<13>{}), token(ITag<14>{}), token(ITag<15>{});
            // (an integer test on the magnitude bits, which an infinity fails.  fmaxf
            // drops a NaN; for finite inputs a NaN sum comes only after one that was
            // infinite or zero, whose z or 1 / z fails the test)
            uint32_t chk_bits = __float_as_uint(chk);
            asm volatile("" : "+v"(chk_bits));
            const bool bad = (chk_bits & 0x7fffffffu) > 0x71800000u;   // 2^100
            if (__builtin_amdgcn_ballot_w64(sact && bad) != 0) {
                // some softmax sum left the range: the chunk again, maximum subtracted
                start();
                rprev = rprev0;
                auto slow = [&](auto tag) {
                    constexpr int t = decltype(tag)::value;
                    load_a(t);
                    const float dd = error(tag, D[t / 4][t % 4]);
                    // (fp32 logits up to the type's limits, masks of its lowest value
                    // among them: log2(e) times the difference from the maximum, not
                    // a difference of products that may have overflowed)
                    const float e = TP ? -kS2 * dd * dd : fmaf(C::SCALED ? -dd : -0.5f * dd, dd, slk[t]);
                    const float em = e - lane_max(sact ? e : -INFINITY);
                    float ex = sact ? __builtin_amdgcn_exp2f(TP || C::SCALED ? em : kLog2e * em) : 0.0f;
                    if constexpr (TP) ex *= fmaf(sgs[t], rprev, slk[t]);
                    const float iz = rcp_fast(lane_sum(ex));
                    const float cs = sact ? sbeta[t] * dd * ex * iz : 0.0f;
                    if constexpr ((t + 2) / 4 != (t + 1) / 4)
                        D[(t + 1) / 4] = __builtin_amdgcn_mfma_f32_4x4x1f32(A[t][(t + 1) / 4], cs,
                                                                            D[(t + 1) / 4], 0, 0, 0);
                    defer(tag, cs);
                    sm.c[gs][scst][t] = C::IS * cs;
                    keep_r(t, ex * iz, dd);
                };
                slow(ITag<0>{}), slow(ITag<1>{}), slow(ITag<2>{}), slow(ITag<3>{});
                slow(ITag<4>{}), slow(ITag<5>{}), slow(ITag<6>{}), slow(ITag<7>{});
                slow(ITag<8>{}), slow(ITag<9>{}), slow(ITag<10>{}), slow(ITag<11>{});
                slow(ITag<12>{}), slow(ITag<13>{}), slow(ITag<14>{}), slow(ITag<15>{});
            }
            block_sync_lds();   // e(n)
            if (n + 1 < NCH) seq_inputs(n + 1);
            block_sync_lds();   // i(n+1)
        }
        block_sync_lds();   // epilogue
        if constexpr (TP) {
            // r of the last token: part 0 of the prior state
            if (sact && a.prior_out)
                a.prior_out[(((size_t)b * H + h) * 2 * J + sj) * Dv + d0 + sdd] = rlast;
        }
    } else if (GT && w >= J + 1 + kGH) {
        if constexpr (HG) {
        // ================= gate waves: two key indices a lane =================
        // E^-1 of chunk n + 2 in phase A of chunk n, from logits loaded a chunk
        // before; its slots were last read in chunk n - 1 (E^-1: chunk n - 1's
        // update operand in phase A; E_C: phase B).
        const int e = 2 * (64 * (w - (J + 1 + kGH)) + lane);   // j * Dk + key index
        const bool act = e < J * DK;
        const int ec = act ? e : 0, gj = ec / DK, gi = ec % DK;
        // two inputs as one word (bf16) or two
        using X2 = typename std::conditional<F32, float2, uint32_t>::type;
        const X2 *const Gg = reinterpret_cast<const X2 *>(
            static_cast<const In *>(a.decay) + ((size_t)b * T * H + h) * J * DK + ec);
        const size_t row = (size_t)H * J * DK / 2;   // one token on
        X2 x[kGC];
        auto lo_of = [](const X2 &v) {
            if constexpr (F32) return v.x;
            else return __uint_as_float(v << 16);
        };
        auto hi_of = [](const X2 &v) {
            if constexpr (F32) return v.y;
            else return __uint_as_float(v & 0xffff0000u);
        };
        auto load = [&](int m) {
#pragma unroll
            for (int t = 0; t < kGC; ++t) x[t] = Gg[(size_t)min(m * kGC + t, T - 1) * row];
        };
        auto gates = [&](int m) {
            const int nt = min(kGC, T - m * kGC), sl = m % 3;
            float f0[kGC], f1[kGC];
            // the running product of 1 + e: in the 24-bit forms in 64 bits (one fused
            // multiply-add, which runs at the rate of a 32-bit one), so that each E^-1 is
            // rounded once and not twice a token
            typename std::conditional<NP == 3, double, float>::type p0 = 1, p1 = 1;
            auto step = [](auto &p, float e) {
                if constexpr (NP == 3) p = fma(p, (double)e, p);
                else p *= 1.0f + e;
                return (float)p;
            };
            float c0 = 1.0f, c1 = 1.0f;
#pragma unroll
            for (int t = 0; t < kGC; ++t) {
                // tokens past the end decay nothing
                const float e0 = __builtin_amdgcn_exp2f(-kLog2e * lo_of(x[t]));
                const float e1 = __builtin_amdgcn_exp2f(-kLog2e * hi_of(x[t]));
                f0[t] = c0 = step(p0, t < nt ? e0 : 0.0f);
                f1[t] = c1 = step(p1, t < nt ? e1 : 0.0f);
            }
            float r0 = rcp_fast(c0), r1 = rcp_fast(c1);
            const bool mine = act && (!(c0 <= kGramEinv) || !(c1 <= kGramEinv));
            // lanes of this component in this wave (a component of 128 key indices
            // fills a wave, one of 64 half a wave, ...)
            const uint64_t all = __builtin_amdgcn_ballot_w64(mine);
            constexpr int CL = DK / 2 < 64 ? DK / 2 : 64;
            const uint64_t cm = CL == 64 ? ~0ull : ((1ull << (CL % 64)) - 1) << (lane / CL * CL);
            const bool deep = (all & cm) != 0;
            if (all != 0 && deep) {
                // deep chunk: the gates, in place of E^-1
                r0 = r1 = 1.0f;
#pragma unroll
                for (int t = 0; t < kGC; ++t) {
                    f0[t] = t < nt ? sigmoid(lo_of(x[t])) : 1.0f;
                    f1[t] = t < nt ? sigmoid(hi_of(x[t])) : 1.0f;
                    r0 *= f0[t], r1 *= f1[t];
                }
            }
            if (act) {
#pragma unroll
                for (int t = 0; t < kGC; ++t)
                    *reinterpret_cast<float2 *>(&sm.ei[sl % C::NEI][gj][t][gi]) = make_float2(f0[t], f1[t]);
                *reinterpret_cast<float2 *>(&sm.ec[sl % C::NEC][gj][gi]) = make_float2(r0, r1);
                if (gi == 0) sm.deep[sl][gj] = deep;
            }
        };
        block_sync_lds();   // prologue 1
        load(0);
        gates(0);
        if (NCH > 1) {
            load(1);
            gates(1);
        }
        if (NCH > 2) load(2);
        block_sync_lds();   // prologue 2
        block_sync_lds();   // prologue 3
        block_sync_lds();   // prologue 4
        for (int n = 0; n < NCH; ++n) {
            if (n + 2 < NCH) {
                gates(n + 2);
                if (n + 3 < NCH) load(n + 3);
            }
            block_sync_lds();   // e(n)
            block_sync_lds();   // i(n+1)
        }
        block_sync_lds();   // epilogue
        }
    } else {
        // ================= helper waves: inputs, priors, outputs =================
        const int bt = 64 * (w - (J + 1)) + lane;
        constexpr int NBT = 64 * kGH;
        // the logits, which are most of the work, are dealt from the first helper
        // wave on, everything else from the second
        const int br = (bt + NBT - 64) % NBT;
        const bool obf = a.out_bf16;
        const In *const Kg = static_cast<const In *>(a.k);
        const In *const Qg = static_cast<const In *>(a.q);
        const In *const Vg = static_cast<const In *>(a.v);
        const In *const LBg = static_cast<const In *>(a.lb);
        const In *const LKg = static_cast<const In *>(a.lk);
        const In *const LQg = static_cast<const In *>(a.lq);
        const uint16_t *const Gg = static_cast<const uint16_t *>(a.decay);
        // one chunk's raw inputs, in registers from fetch to land
        constexpr int E = C::E;
        constexpr int NKQ = ceil_div_c(kGC * DK / E, NBT);   // uint4 of K (and of Q)
        constexpr int NLG = ceil_div_c(kGC * N / E, NBT);    // uint4 of each logit tensor
        constexpr int NV = ceil_div_c(kGC * DB / E, NBT);
        constexpr int NG = HG || !GT ? 1 : ceil_div_c(kGC * J * DK / 8, NBT);   // uint4 of the decay logits
        uint4 rk[NKQ], rq[NKQ], rlb[NLG], rlk[NLG], rlq[NLG], rv[NV], rg[NG];
        uint4 rgk[TP ? NV : 1], rgq[TP ? NV : 1];   // temporal: the gate logits
        // Every thread loads every item it owns, from a clamped row (the last
        // token of the chunk, the last item): the loads go out back to back,
        // with no branch each.  land() zeroes what lies past the end, a phase
        // later, so that nothing here waits for the data.
        auto fetch = [&](int m) {
            const int t0 = m * kGC, nt = min(kGC, T - t0);
            const size_t row0 = (size_t)b * T + t0;
#pragma unroll
            for (int x = 0; x < NKQ; ++x) {
                const int e = min(br + NBT * x, kGC * DK / E - 1);
                const int t = min(e / (DK / E), nt - 1), p = e % (DK / E);
                const size_t off = ((row0 + t) * H + h) * DK + E * p;
                rk[x] = *reinterpret_cast<const uint4 *>(Kg + off);
                rq[x] = *reinterpret_cast<const uint4 *>(Qg + off);
            }
#pragma unroll
            for (int x = 0; x < NLG; ++x) {
                const int e = min(bt + NBT * x, kGC * N / E - 1);
                const int t = min(e / (N / E), nt - 1), rem = e % (N / E);
                const int j = rem / (DB / E), p = rem % (DB / E);
                const size_t off = (((row0 + t) * H + h) * J + j) * Dv + d0 + E * p;
                rlb[x] = *reinterpret_cast<const uint4 *>(LBg + off);
                rlk[x] = *reinterpret_cast<const uint4 *>(LKg + off);
                rlq[x] = *reinterpret_cast<const uint4 *>(LQg + off);
            }
#pragma unroll
            for (int x = 0; x < NV; ++x) {
                const int e = min(br + NBT * x, kGC * DB / E - 1);
                const int t = min(e / (DB / E), nt - 1), p = e % (DB / E);
                const size_t off = ((row0 + t) * H + h) * Dv + d0 + E * p;
                rv[x] = *reinterpret_cast<const uint4 *>(Vg + off);
                if constexpr (TP) {
                    rgk[x] = *reinterpret_cast<const uint4 *>(static_cast<const In *>(a.gk) + off);
                    rgq[x] = *reinterpret_cast<const uint4 *>(static_cast<const In *>(a.gq) + off);
                }
            }
            if constexpr (GT && !HG)
#pragma unroll
            for (int x = 0; x < NG; ++x) {
                const int e = min(bt + NBT * x, kGC * J * DK / 8 - 1);
                const int t = min(e / (J * DK / 8), nt - 1), p = e % (J * DK / 8);
                rg[x] = *reinterpret_cast<const uint4 *>(Gg + ((row0 + t) * H + h) * J * DK + E * p);
            }
        };
        // r, or zero when !keep (a mask: a select of the whole vector would be
        // made on addresses and put the registers in scratch memory)
        auto mask4 = [](const uint4 &r, bool keep) {
            const uint32_t m = keep ? 0xffffffffu : 0u;
            return make_uint4(r.x & m, r.y & m, r.z & m, r.w & m);
        };
        // chunk m's inputs but its decay logits to its slot
        auto land = [&](int m) {
            const int s3 = m % 3, nt = min(kGC, T - m * kGC);
#pragma unroll
            for (int x = 0; x < NKQ; ++x) {
                const int e = br + NBT * x, t = e / (DK / E), p = e % (DK / E);
                if (e < kGC * DK / E) {
                    // rows past the end are zero; bf16: two 8-byte stores (the
                    // padded rows are 8-byte aligned)
                    const uint4 kk = mask4(rk[x], t < nt), qq = mask4(rq[x], t < nt);
                    if constexpr (F32) {
                        *reinterpret_cast<uint4 *>(&sm.k[s3][t][E * p]) = kk;
                        *reinterpret_cast<uint4 *>(&sm.q[s3][t][E * p]) = qq;
                    } else {
                        uint2 *dk = reinterpret_cast<uint2 *>(&sm.k[s3][t][E * p]);
                        uint2 *dq = reinterpret_cast<uint2 *>(&sm.q[s3][t][E * p]);
                        dk[0] = make_uint2(kk.x, kk.y);
                        dk[1] = make_uint2(kk.z, kk.w);
                        dq[0] = make_uint2(qq.x, qq.y);
                        dq[1] = make_uint2(qq.z, qq.w);
                    }
                }
            }
            // query-prior logits to the slot; beta = sigmoid(beta logit) and the
            // key-prior logits, and v, straight to the sequential wave's arrays
            // (chunk m's pair of them was last read in phase B of chunk m - 3)
#pragma unroll
            for (int x = 0; x < NLG; ++x) {
                const int e = bt + NBT * x, t = e / (N / E), colE = E * (e % (N / E));
                if (e < kGC * N / E) {
                    const bool in = t < nt;
                    *reinterpret_cast<uint4 *>(&sm.lq[s3][t][colE]) = mask4(rlq[x], in);
#pragma unroll
                    for (int y = 0; y < E; ++y) {
                        const float xb = piece<F32>(rlb[x], y), xk = piece<F32>(rlk[x], y);
                        // (temporal: key_priors forms the second value)
                        if constexpr (TP)
                            sm.sq[m & 1][colE + y][t].x = in ? sigmoid(xb) : 0.0f;
                        else
                            sm.sq[m & 1][colE + y][t] =
                                make_float2(in ? sigmoid(xb) : 0.0f, !in ? 0.0f : C::SCALED ? kLog2e * xk : xk);
                    }
                    if constexpr (TP)
                        *reinterpret_cast<uint4 *>(&sm.lk[m & 1][t][colE]) = mask4(rlk[x], in);
                }
            }
#pragma unroll
            for (int x = 0; x < NV; ++x) {
                const int e = br + NBT * x, t = e / (DB / E), p = e % (DB / E);
                if (e < kGC * DB / E) {
#pragma unroll
                    for (int y = 0; y < E; ++y) {
                        sm.vs[m & 1][E * p + y][t] = t < nt ? C::S * piece<F32>(rv[x], y) : 0.0f;
                        if constexpr (TP) {
                            // (tokens past the end keep both priors; key_priors turns
                            // the first into 1 - g^k)
                            sm.gs[m & 1][E * p + y][t] = t < nt ? sigmoid(piece<F32>(rgk[x], y)) : 0.0f;
                            sm.gq[m % 3][t][E * p + y] = t < nt ? sigmoid(piece<F32>(rgq[x], y)) : 0.0f;
                        }
                    }
                }
            }
        };
        // chunk m's decay logits, once the tile waves have taken chunk m - 1's
        auto land_g = [&](int m) {
            const int nt = min(kGC, T - m * kGC);
#pragma unroll
            for (int x = 0; x < NG; ++x) {
                const int e = bt + NBT * x, t = e / (J * DK / 8), p = e % (J * DK / 8);
                if (e < kGC * J * DK / 8)
                    *reinterpret_cast<uint4 *>(&sm.g[t][E * p]) = mask4(rg[x], t < nt);
            }
        };
        // pi^q of chunk m: softmax over j of the query-prior logits, per (t, dd)
        auto priors = [&](int m) {
            const int s3 = m % 3;
            for (int e = br; e < kGC * DB; e += NBT) {
                const int t = e / DB, dd = e % DB;
                float x[J], mx = -INFINITY, z = 0.0f;
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    x[j] = bf(sm.lq[s3][t][j * DB + dd]);
                    mx = fmaxf(mx, x[j]);
                }
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    x[j] = __builtin_amdgcn_exp2f(kLog2e * (x[j] - mx));
                    z += x[j];
                }
                const float iz = rcp_fast(z);
#pragma unroll
                for (int j = 0; j < J; ++j) sm.pq[m & 1][t][j * DB + dd] = J == 1 ? 1.0f : x[j] * iz;
            }
        };
        // temporal: g^k pi^k and 1 - g^k of chunk m, pi^k = softmax over j of the key-prior logits
        auto key_priors = [&](int m) {
            for (int e = br; e < kGC * DB; e += NBT) {
                const int t = e % kGC, dd = e / kGC;
                float x[J], mx = -INFINITY, z = 0.0f;
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    x[j] = bf(sm.lk[m & 1][t][j * DB + dd]);
                    mx = fmaxf(mx, x[j]);
                }
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    x[j] = __builtin_amdgcn_exp2f(kLog2e * (x[j] - mx));
                    z += x[j];
                }
                const float g = sm.gs[m & 1][dd][t], f = g * rcp_fast(z);
                sm.gs[m & 1][dd][t] = 1.0f - g;
#pragma unroll
                for (int j = 0; j < J; ++j) sm.sq[m & 1][j * DB + dd][t].y = f * x[j];
            }
        };
        // temporal: the running query prior rhobar over chunk m in place of pi^q, one
        // thread per column (the last N), carried from chunk to chunk
        const int qc = bt - (NBT - N);
        float rho = 1.0f / J;
        if constexpr (TP) {
            if (qc >= 0 && a.prior_in)
                rho = a.prior_in[(((size_t)b * H + h) * 2 * J + J + qc / DB) * Dv + d0 + qc % DB];
        }
        auto scan_prior = [&](int m) {
            if (qc >= 0) {
                float pi[kGC], g[kGC];
#pragma unroll
                for (int t = 0; t < kGC; ++t) pi[t] = sm.pq[m & 1][t][qc], g[t] = sm.gq[m % 3][t][qc % DB];
#pragma unroll
                for (int t = 0; t < kGC; ++t) pi[t] = rho = fmaf(g[t], pi[t] - rho, rho);
#pragma unroll
                for (int t = 0; t < kGC; ++t) sm.pq[m & 1][t][qc] = pi[t];
            }
        };
        // output of chunk m: o = sum_j pi^q y
        auto output = [&](int m) {
            if (AX && !a.o) return;
            const int mt0 = m * kGC, nt = min(kGC, T - mt0);
            for (int e = br; e < kGC * DB; e += NBT) {
                const int t = e / DB, dd = e % DB;
                if (t >= nt) continue;
                float o = 0.0f;
#pragma unroll
                for (int j = 0; j < J; ++j) o += sm.py[m & 1][t][j * DB + dd];
                store1(a.o, (((size_t)b * T + mt0 + t) * H + h) * Dv + d0 + dd, o, obf);
            }
        };

        block_sync_lds();   // prologue 1
        fetch(0);
        land(0);
        if constexpr (GT && !HG) land_g(0);
        if (NCH > 1) {
            fetch(1);
            land(1);
        }
        block_sync_lds();   // prologue 2
        if constexpr (TP) {
            key_priors(0);
            if (NCH > 1) key_priors(1);
        }
        block_sync_lds();   // prologue 3: the tile waves have read chunk 0's decay logits
        if constexpr (GT && !HG)
            if (NCH > 1) land_g(1);
        if (NCH > 2) fetch(2);
        block_sync_lds();   // prologue 4
        for (int n = 0; n < NCH; ++n) {
            priors(n);
            if (n >= 2) output(n - 2);
            // chunk n + 2 lands in the slots of chunk n - 1
            if (n + 2 < NCH) land(n + 2);
            block_sync_lds();   // e(n)
            // its decay logits in phase B, when those of chunk n + 1 have been read
            if constexpr (GT && !HG)
                if (n + 2 < NCH) land_g(n + 2);
            if constexpr (TP) {
                scan_prior(n);
                if (n + 2 < NCH) key_priors(n + 2);
            }
            if (n + 3 < NCH) fetch(n + 3);
            block_sync_lds();   // i(n+1)
        }
        if (NCH >= 2) output(NCH - 2);
        block_sync_lds();   // epilogue
        output(NCH - 1);
        if constexpr (TP) {
            // the running query prior after the last token: part 1 of the prior state
            if (qc >= 0 && a.prior_out)
                a.prior_out[(((size_t)b * H + h) * 2 * J + J + qc / DB) * Dv + d0 + qc % DB] = rho;
        }
    }
}

template <int DK, int J, int DB, bool TP, bool GT, bool F32>
hipError_t launch_g(const LayerArgs &a, hipStream_t stream) {
    using C = GCfg<DK, J, DB, TP, GT, F32>;
    const long blocks = (long)(a.Dv / DB) * a.H * a.B;
    hipLaunchKernelGGL((scan_gated_chunk_kernel<DK, J, DB, TP, GT, F32>), dim3((unsigned)blocks),
                       dim3(64 * C::NWAVE), 0, stream, a);
    return hipGetLastError();
}

template <int DK, int J, bool TP, bool GT, bool F32>
hipError_t launch_gj(const LayerArgs &a, hipStream_t stream) {
    if constexpr (J * DK > (TP || F32 ? 256 : 384)) {
        return hipErrorInvalidValue;
    } else {
        // 16 output dims per block once that grid fills the chip (where their LDS
        // fits: fp32 inputs with gates and temporal priors at J * Dk = 256 do not);
        // 8 below
        static_assert(sizeof(GSmem<DK, J, 8, TP, GT, F32>) <= 160 * 1024, "LDS");
        if constexpr (sizeof(GSmem<DK, J, 16, TP, GT, F32>) <= 160 * 1024)
            if (a.Dv % 16 == 0 && (long)(a.Dv / 16) * a.H * a.B >= 256)
                return launch_g<DK, J, 16, TP, GT, F32>(a, stream);
        return launch_g<DK, J, 8, TP, GT, F32>(a, stream);
    }
}

template <int DK, bool TP, bool GT, bool F32>
hipError_t launch_gdk(const LayerArgs &a, hipStream_t stream) {
    switch (a.J) {
        case 1: return launch_gj<DK, 1, TP, GT, F32>(a, stream);
        case 2: return launch_gj<DK, 2, TP, GT, F32>(a, stream);
        case 3: return launch_gj<DK, 3, TP, GT, F32>(a, stream);
        case 4: return launch_gj<DK, 4, TP, GT, F32>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

template <bool TP, bool GT, bool F32>
hipError_t launch_gated(const LayerArgs &a, hipStream_t stream) {
    switch (a.Dk) {
        case 16: return launch_gdk<16, TP, GT, F32>(a, stream);
        case 32: return launch_gdk<32, TP, GT, F32>(a, stream);
        case 64: return launch_gdk<64, TP, GT, F32>(a, stream);
        case 128: return launch_gdk<128, TP, GT, F32>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace
}  // namespace swila
