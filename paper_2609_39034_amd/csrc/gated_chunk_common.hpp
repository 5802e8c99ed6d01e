// What the two chunk kernels of the gated forms share (scan_gated_chunk_kernel.hpp,
// scan_gated_chunk_wide.hip): products of fp32 operands in bf16 parts, the block order,
// and the products of a deep chunk.
#pragma once

#include "device_common.hpp"

namespace swila {
namespace {

typedef short short4v __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kGC = 16;              // tokens per chunk
constexpr float kGramEinv = 2.35385266837019985e17f;   // e^40: factorised Gram products while every E^-1 <= this
// The sequential wave works in scaled units: with s^2 = log2(e) / 2, d = s (v - pred)
// makes the E-step exponent log2(e) (lk - delta^2 / 2) a single fused multiply-add,
// -d * d + log2(e) lk, and the coefficient s c = beta r d feeds s pred.
constexpr float kS = 0.84932180028801904272f;      // sqrt(log2(e) / 2)
constexpr float kInvS = 1.17741002251547469101f;   // 1 / kS
constexpr float kS2 = 0.72134752044448170368f;     // kS^2
constexpr int ceil_div_c(int x, int y) { return (x + y - 1) / y; }

__device__ __forceinline__ floatx4 mfma16(short4v a, short4v b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Four fp32 values as P bf16 parts each: a high part (round to nearest) and P - 1
// residuals, converted two at a time.  Two parts are good to about 2^-17 of the
// value, three to all of its 24 bits.
template <int P>
struct S4 {
    short4v x[P];
};
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
template <int P>
__device__ __forceinline__ void split2(float a, float b, uint32_t (&o)[P]) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
        o[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2v));
        a -= __uint_as_float(o[p] << 16);
        b -= __uint_as_float(o[p] & 0xffff0000u);
    }
}
template <int P>
__device__ __forceinline__ S4<P> split4(float x0, float x1, float x2, float x3) {
    uint32_t u[P], v[P];
    split2<P>(x0, x1, u);
    split2<P>(x2, x3, v);
    S4<P> s;
#pragma unroll
    for (int p = 0; p < P; ++p) s.x[p] = __builtin_bit_cast(short4v, make_uint2(u[p], v[p]));
    return s;
}
template <int P>
__device__ __forceinline__ S4<P> split4(floatx4 x) { return split4<P>(x[0], x[1], x[2], x[3]); }
template <int P>
__device__ __forceinline__ S4<P> zero4() {
    S4<P> s;
#pragma unroll
    for (int p = 0; p < P; ++p) s.x[p] = short4v{0, 0, 0, 0};
    return s;
}
// a b with both operands split: the products of parts p and r with p + r < P
// (hi hi + hi lo + lo hi; with three parts six products, dropping about 2^-26).
// With three parts the small products are summed apart, smallest first, so that
// acc is rounded twice and not six times.
template <int P, typename V, typename M>
__device__ __forceinline__ floatx4 mm_parts(const V (&a)[P], const V (&b)[P], floatx4 acc, M &&mul) {
    if constexpr (P == 3) {
        floatx4 lo = mul(a[2], b[0], floatx4{0.f, 0.f, 0.f, 0.f});
        lo = mul(a[1], b[1], lo);
        lo = mul(a[0], b[2], lo);
        lo = mul(a[1], b[0], lo);
        lo = mul(a[0], b[1], lo);
        return mul(a[0], b[0], acc) + lo;
    } else {
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int r = 0; r < P - p; ++r) acc = mul(a[p], b[r], acc);
        return acc;
    }
}
template <int P>
__device__ __forceinline__ floatx4 mm(const S4<P> &a, const S4<P> &b, floatx4 acc) {
    return mm_parts<P>(a.x, b.x, acc, [](short4v x, short4v y, floatx4 c) { return mfma16(x, y, c); });
}
// The same over two 16-wide k tiles at once (a0 b0 + a1 b1), on the 32-deep
// instruction: a lane's eight k elements are its four of tile 0, then its four
// of tile 1, in both operands.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ bf16x8 join8(short4v x, short4v y) {
    return __builtin_bit_cast(bf16x8, make_uint4(__builtin_bit_cast(uint2, x).x,
                                                 __builtin_bit_cast(uint2, x).y,
                                                 __builtin_bit_cast(uint2, y).x,
                                                 __builtin_bit_cast(uint2, y).y));
}
template <int P>
__device__ __forceinline__ floatx4 mmx2(const S4<P> &a0, const S4<P> &a1, const S4<P> &b0,
                                        const S4<P> &b1, floatx4 acc) {
    bf16x8 a[P], b[P];
#pragma unroll
    for (int p = 0; p < P; ++p) a[p] = join8(a0.x[p], a1.x[p]), b[p] = join8(b0.x[p], b1.x[p]);
    return mm_parts<P>(a, b, acc, [](bf16x8 x, bf16x8 y, floatx4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, c, 0, 0, 0);
    });
}

__device__ __forceinline__ float bf(float x) { return x; }   // (an fp32 input as it is)
__device__ __forceinline__ float bf(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// four consecutive inputs of an LDS row
__device__ __forceinline__ float4 in4(const uint16_t *p) {
    const uint2 r = *reinterpret_cast<const uint2 *>(p);
    return make_float4(__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u),
                       __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u));
}
__device__ __forceinline__ float4 in4(const float *p) { return *reinterpret_cast<const float4 *>(p); }

// Block -> (column block, head): the column blocks of a head on one XCD
// (workgroups go to the eight XCDs round-robin by index, each with its own L2),
// so that the head's K, Q and gate rows are fetched from HBM once.
__device__ __forceinline__ void gated_coords(int id, int ndb, int nheads, int &db, int &head) {
    if (nheads % 8 == 0) {
        const int k = id / 8;
        head = id % 8 + 8 * (k / ndb);
        db = k % ndb;
    } else {
        head = id / ndb;
        db = id % ndb;
    }
}

template <int V>
struct ITag {
    static constexpr int value = V;
};

// ---- Deep chunks: those over which some gates decay past the range of the factorised
// products (E^-1 above kGramEinv), a gate that is closed altogether (a = 0) among
// them.  A holds the gates themselves, A[t][i] = a_t,i (1 past the sequence's end), and
// every factor is the product of the gates that it stands for: never a difference of
// cumulative logarithms, which loses the later gates behind a strongly closed one
// (relative 2e-5 behind a logit of -50, all of them behind -1e9) and is inf - inf
// behind a gate of 0.
//
// Lane (tl, lg) holds token t = tl.  Over the aligned blocks of 2^l tokens: p = the
// gates from the start of t's block up to t, s = those after t up to the block's
// end, all = the whole block's.  One step doubles the blocks; the other half's product is
// the same in all of its lanes, so that mirrored rows fetch it.
struct Span4 {
    float p[4], s[4], all[4];
    __device__ __forceinline__ explicit Span4(const float4 &a)
        : p{a.x, a.y, a.z, a.w}, s{1.f, 1.f, 1.f, 1.f}, all{a.x, a.y, a.z, a.w} {}
    template <int L>
    __device__ __forceinline__ void grow(bool upper) {
        constexpr int CTRL = L == 0 ? 0xb1 : L == 1 ? 0x4e : L == 2 ? 0x141 : 0x140;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const float o = dpp_mov<CTRL>(all[x]);
            p[x] *= upper ? o : 1.0f;
            s[x] *= upper ? 1.0f : o;
            all[x] *= o;
        }
    }
};
// E at token tl for key indices i .. i + 3: the gates of tokens 0 .. tl
template <int LP>
__device__ __forceinline__ float4 decay_to(const float (*A)[LP], int tl, int i) {
    asm volatile("" : "+v"(tl));   // (as in deep_grams)
    Span4 a(*reinterpret_cast<const float4 *>(&A[tl][i]));
    a.template grow<0>(tl & 1);
    a.template grow<1>(tl & 2);
    a.template grow<2>(tl & 4);
    a.template grow<3>(tl & 8);
    return make_float4(a.p[0], a.p[1], a.p[2], a.p[3]);
}
// E_C / E at tokens 4 lg + m, m = 0 .. 3, for key index i: the gates of the chunk's
// tokens after them
template <int LP>
__device__ __forceinline__ void decay_after(const float (*A)[LP], int lg, int i, float (&f)[4]) {
    float p = 1.0f;
    asm volatile("" : "+v"(lg));   // (as in deep_grams)
#pragma unroll
    for (int u = kGC - 1; u >= 0; --u) {
        f[u % 4] = lg == u / 4 ? p : f[u % 4];
        p *= A[u][i];
    }
}
// g[r] = sum_i K[t][i] K[s][i] (a_{s+1} .. a_t)_i at t = 4 lg + r, s = tl (0 for t <= s),
// qg[r] = sum_i Q[t][i] K[s][i] (a_{s+1} .. a_t)_i at t = tl, s = 4 lg + r (0 for s > t).
// Tokens s < t whose highest different bit is l lie in the lower and the upper
// half of one block of 2^(l+1): the factor is s's product up to the middle times t's
// from there, so one product per l of rows scaled by either gives all such pairs
// (its other entries are not used).
// With every chunk deep, B=4 H=8 T=512, against each pair's factor by itself from
// cumulative logarithms: bf16 D=64 J=4 1.06 -> 0.21 ms, fp32 1.00 -> 0.28 (the token
// scan 0.29), fp32 Dk=128 Dv=64 J=2 1.92 -> 0.51 (the token scan 0.24: the one range
// where that stays ahead).  One key tile a step: two would be 15 to 20% faster here,
// but the registers that they take went to scratch memory around the open-gate path
// (D=64 J=4 with temporal priors 109 -> 118 us).
template <int DK, int P, int LP, int KP, typename In>
__device__ __forceinline__ void deep_grams(const float (*A)[LP], const In (*K)[KP], const In (*Q)[KP],
                                           int tl, int lg, floatx4 &g, floatx4 &qg) {
    // (the lane masks below belong to this rare path alone: kept from the compiler's
    // hoisting them out of the chunk loop, where they would hold registers)
    asm volatile("" : "+v"(tl), "+v"(lg));
    const floatx4 zero = floatx4{0.f, 0.f, 0.f, 0.f};
    floatx4 gl[4] = {zero, zero, zero, zero}, ql[5] = {zero, zero, zero, zero, zero};
#pragma unroll 1
    for (int i0 = 0; i0 < DK; i0 += 16) {
        const float4 k = in4(&K[tl][i0 + 4 * lg]), q = in4(&Q[tl][i0 + 4 * lg]);
        Span4 a(*reinterpret_cast<const float4 *>(&A[tl][i0 + 4 * lg]));
        S4<P> kx = split4<P>(k.x, k.y, k.z, k.w), qx = split4<P>(q.x, q.y, q.z, q.w);
        ql[4] = mm<P>(kx, qx, ql[4]);   // t = s: D[4 lg + r][tl]
        auto level = [&](auto tag) {
            constexpr int L = decltype(tag)::value;
            const bool upper = (tl >> L) & 1;
            float f[4];
#pragma unroll
            for (int y = 0; y < 4; ++y) f[y] = upper ? a.p[y] : a.s[y];
            kx = split4<P>(k.x * f[0], k.y * f[1], k.z * f[2], k.w * f[3]);
            qx = split4<P>(q.x * f[0], q.y * f[1], q.z * f[2], q.w * f[3]);
            a.template grow<L>(upper);
            gl[L] = mm<P>(kx, kx, gl[L]);   // D[t = 4 lg + r][s = tl]
            ql[L] = mm<P>(kx, qx, ql[L]);   // D[s = 4 lg + r][t = tl]
        };
        level(ITag<0>{}), level(ITag<1>{}), level(ITag<2>{}), level(ITag<3>{});
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = 4 * lg + r, x = o ^ tl;   // the other token
        const float gv = x >= 8 ? gl[3][r] : x >= 4 ? gl[2][r] : x >= 2 ? gl[1][r] : gl[0][r];
        const float qv = x >= 8 ? ql[3][r] : x >= 4 ? ql[2][r] : x >= 2 ? ql[1][r] : x == 1 ? ql[0][r] : ql[4][r];
        g[r] = o > tl ? gv : 0.0f;
        qg[r] = o <= tl ? qv : 0.0f;
    }
}

}  // namespace
}  // namespace swila
