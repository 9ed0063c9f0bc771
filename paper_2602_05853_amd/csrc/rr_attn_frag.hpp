// Operand fragments of attention on 16 x 16 matrix tiles, straight from global memory to registers (rr_attn_generic.hip,
// rr_attn_decode.hip).
//
// Transposed products, S^T = K Q^T and O^T = V^T P^T: a lane owns one query (column lane % 16), and the accumulator
// layout of S^T (keys 4 (lane / 16) + 0..3 of a tile) is the B operand of the second product.  V^T fragments need
// consecutive keys of one channel per lane; which channel a lane's row stands for is free, so lane x = lane % 16 loads
// W consecutive channels W x .. W x + W - 1 of each of its keys and these W values belong to W different tiles: with
// fp32 they are the fragments as loaded, with bf16 one byte permutation per register pairs two keys.
//
// Values that are not finite.  A product of tiles also multiplies what a row does not take: probabilities of zero (keys
// behind the end of a block, blocks of another row's list) and the zero terms of a split probability.  Zero times
// infinity is not a number, and sums keep that, so a wave that finds one in its result (has_nan) takes its keys once more with
// such values left out (kCareful).  Checking every value as it is loaded was vector work on every key.
#pragma once
#include "rr_common.hpp"

#include <type_traits>

namespace rr {

namespace {

constexpr float kFragLazySum = 256.0f;               // a step's sum of exponentials above it moves the softmax reference

// f(W, base) for every piece of a row of 16 NT channels that a lane loads at once: W channels, lane x those from
// base + W x on
template <int WMAX, int NT, typename F>
__device__ __forceinline__ void for_pieces(F&& f) {
    using std::integral_constant;
    constexpr int full = NT / WMAX;
    if constexpr (full > 0) f(integral_constant<int, WMAX>{}, integral_constant<int, 0>{});
    if constexpr (full > 1) f(integral_constant<int, WMAX>{}, integral_constant<int, 16 * WMAX>{});
    if constexpr (full > 2) f(integral_constant<int, WMAX>{}, integral_constant<int, 32 * WMAX>{});
    if constexpr (full > 3) f(integral_constant<int, WMAX>{}, integral_constant<int, 48 * WMAX>{});
    static_assert(full <= 4, "at most 256 channels");
    constexpr int r8 = WMAX * full;
    if constexpr (WMAX > 4 && ((NT - r8) & 4)) f(integral_constant<int, 4>{}, integral_constant<int, 16 * r8>{});
    constexpr int r4 = r8 + (WMAX > 4 ? ((NT - r8) & 4) : 0);
    if constexpr ((NT - r4) & 2) f(integral_constant<int, 2>{}, integral_constant<int, 16 * r4>{});
    constexpr int r2 = r4 + ((NT - r4) & 2);
    if constexpr ((NT - r2) & 1) f(integral_constant<int, 1>{}, integral_constant<int, 16 * r2>{});
}

// Fragments of one element type for rows of up to 16 NT channels.
//   KF   K (or Q) operand of one 16-row tile: this lane's channels of row lane % 16
//   VF   V^T operand of one pair of tiles (32 keys): this lane's 8 keys
template <typename T, int NT, int TL> struct Frag;

template <int NT, int TL> struct Frag<float, NT, TL> {
    static constexpr int kW = 4;
    f32x4 k[NT];                                     // chunk i: channels 16 i + 4 g .. +3
    struct V { float v[4 * TL][NT]; };                    // [tile * 4 + r][channel tile]

    __device__ __forceinline__ void load(const float* row, int d, int gq) {
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int c = 16 * i + 4 * gq;
            if (i < NT - 1) {
                k[i] = *reinterpret_cast<const f32x4*>(row + c);
            } else {
                const bool in = c < d;                // channels that do not exist are zero on both sides
                const f32x4 v = *reinterpret_cast<const f32x4*>(row + (in ? c : 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) k[i][e] = in ? v[e] : 0.f;
            }
        }
    }
    __device__ static __forceinline__ void load_v(V& o, int key, const float* row, int d, int x) {
        for_pieces<kW, NT>([&](auto w, auto base) {
            constexpr int W = decltype(w)::value, B0 = decltype(base)::value;
            const int c = min(B0 + W * x, d - W);     // channels past d are never stored
            typedef __attribute__((ext_vector_type(W))) float vec;
            if constexpr (W == 1) {
                o.v[key][B0 / 16] = row[c];
            } else {
                const vec v = *reinterpret_cast<const vec*>(row + c);
#pragma unroll
                for (int e = 0; e < W; ++e) o.v[key][B0 / 16 + e] = v[e];
            }
        });
    }
    // scores of the two tiles of a pair; interleaved so that consecutive MFMAs do not depend on each other
    template <int QT>
    __device__ static __forceinline__ void qk(f32x4 (&s)[QT][TL], const Frag (&kf)[TL], const Frag (&qf)[QT]) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < TL; ++t)
#pragma unroll
                    for (int u = 0; u < QT; ++u)
                        s[u][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t].k[i][e], qf[u].k[i][e], s[u][t], 0, 0, 0);
    }
    // the values of key slot `key` where `gone`: zero
    __device__ static __forceinline__ void drop(V& v, int key, bool gone) {
#pragma unroll
        for (int t = 0; t < NT; ++t) v.v[key][t] = gone ? 0.f : v.v[key][t];
    }
    template <int QT, bool kCareful>
    __device__ static __forceinline__ void pv(f32x4 (&acc)[QT][NT], const V& v, const float (&p)[QT][4 * TL]) {
#pragma unroll
        for (int key = 0; key < 4 * TL; ++key)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int u = 0; u < QT; ++u)
                    acc[u][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(v.v[key][t], p[u][key], acc[u][t], 0, 0, 0);
    }
};

template <int NT, int TL> struct Frag<bf16_t, NT, TL> {
    static_assert(TL == 2, "the second product takes 32 keys");
    static constexpr int kW = 8;
    static constexpr int KC = (NT + 1) / 2;
    u32x4 k[KC];                                     // chunk i: channels 32 i + 8 g .. +7
    struct V { unsigned v[8][(NT + 1) / 2]; };       // [tile * 4 + r]: the channels as loaded, two to a register

    __device__ __forceinline__ void load(const bf16_t* row, int d, int gq) {
#pragma unroll
        for (int i = 0; i < KC; ++i) {
            const int c = 32 * i + 8 * gq;
            if (i < KC - 1) {
                k[i] = *reinterpret_cast<const u32x4*>(row + c);
            } else {
                const bool in = c < d;
                const u32x4 v = *reinterpret_cast<const u32x4*>(row + (in ? c : 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) k[i][e] = in ? v[e] : 0u;
            }
        }
    }
    __device__ static __forceinline__ void load_v(V& o, int key, const bf16_t* row, int d, int x) {
        for_pieces<kW, NT>([&](auto w, auto base) {
            constexpr int W = decltype(w)::value, B0 = decltype(base)::value;
            const int c = min(B0 + W * x, d - W);
            if constexpr (W == 1) {
                o.v[key][B0 / 32] = row[c].bits;
            } else if constexpr (W == 2) {
                o.v[key][B0 / 32] = *reinterpret_cast<const unsigned*>(row + c);
            } else {
                typedef __attribute__((ext_vector_type(W / 2))) unsigned vec;
                const vec v = *reinterpret_cast<const vec*>(row + c);
#pragma unroll
                for (int e = 0; e < W / 2; ++e) o.v[key][B0 / 32 + e] = v[e];
            }
        });
    }
    template <int QT>
    __device__ static __forceinline__ void qk(f32x4 (&s)[QT][TL], const Frag (&kf)[TL], const Frag (&qf)[QT]) {
#pragma unroll
        for (int i = 0; i < KC; ++i)
#pragma unroll
            for (int t = 0; t < TL; ++t)
#pragma unroll
                for (int u = 0; u < QT; ++u)
                    s[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[t].k[i]),
                                                                      __builtin_bit_cast(bf16x8, qf[u].k[i]), s[u][t], 0, 0, 0);
    }
    __device__ static __forceinline__ void drop(V& v, int key, bool gone) {
#pragma unroll
        for (int i = 0; i < (NT + 1) / 2; ++i) v.v[key][i] = gone ? 0u : v.v[key][i];
    }
    // kCareful: the lower two terms, which may be zero where the probability is not, take finite values only
    template <int QT, bool kCareful>
    __device__ static __forceinline__ void pv(f32x4 (&acc)[QT][NT], const V& v, const float (&p)[QT][4 * TL]) {
        // p = hi + mid + lo, every term the leading 8 significant bits of what is left (truncated, so exact)
        u32x4 plane[QT][3];
#pragma unroll
        for (int u = 0; u < QT; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                unsigned a = __float_as_uint(p[u][2 * j]), b = __float_as_uint(p[u][2 * j + 1]);
                float ra = p[u][2 * j], rb = p[u][2 * j + 1];
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) {
                    plane[u][pl][j] = __builtin_amdgcn_perm(b, a, 0x07060302u);
                    if (pl < 2) {
                        ra -= __uint_as_float(a & 0xFFFF0000u);
                        rb -= __uint_as_float(b & 0xFFFF0000u);
                        a = __float_as_uint(ra);
                        b = __float_as_uint(rb);
                    }
                }
            }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            u32x4 vt;                                // 8 keys of this lane's channel of tile t
            const unsigned sel = (t & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
            for (int j = 0; j < 4; ++j) vt[j] = __builtin_amdgcn_perm(v.v[2 * j + 1][t / 2], v.v[2 * j][t / 2], sel);
            u32x4 vf = vt;
            if (kCareful) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {        // an exponent of all ones carries into the sign's place
                    const unsigned bad = ((vt[j] & 0x7F807F80u) + 0x00800080u) & 0x80008000u;
                    vf[j] = vt[j] & ~(bad | (bad - (bad >> 15)));
                }
            }
#pragma unroll
            for (int pl = 2; pl >= 0; --pl)          // the small terms first
#pragma unroll
                for (int u = 0; u < QT; ++u)
                    acc[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pl > 0 ? vf : vt),
                                                                        __builtin_bit_cast(bf16x8, plane[u][pl]), acc[u][t], 0, 0, 0);
        }
    }
};

// Softmax of one step for the lane's query of one query tile: p = exp2(s scale - ref), sums, and (rarely, the whole wave)
// the reference moved up to the new maximum with the accumulators rescaled.  TL tiles of 16 keys.
template <int TL, int NT>
__device__ __forceinline__ void frag_softmax(const f32x4 (&s)[TL], float scale_log2, float& ref, float& lsum,
                                             f32x4 (&acc)[NT], float (&p)[4 * TL]) {
    const float NEG_INF = -__builtin_huge_valf();
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4 * TL; ++i) {
        p[i] = __builtin_amdgcn_exp2f(fmaf(s[i >> 2][i & 3], scale_log2, -ref));
        sum += p[i];
    }
    // (a reference of -inf, nothing seen yet, gives inf or nan and lands here as well)
    if (__any(!(sum <= kFragLazySum))) {
        float mx = NEG_INF;
#pragma unroll
        for (int i = 0; i < 4 * TL; ++i) mx = fmaxf(mx, s[i >> 2][i & 3]);
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float nref = fmaxf(ref, mx * scale_log2);
        const float use = nref == NEG_INF ? 0.f : nref;
        const float alpha = __builtin_amdgcn_exp2f(ref - use);                  // 0 while the reference is -inf
        ref = nref;
        lsum *= alpha;
#pragma unroll
        for (int c = 0; c < NT; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[c][r] *= alpha;
        sum = 0.f;
#pragma unroll
        for (int i = 0; i < 4 * TL; ++i) {
            p[i] = __builtin_amdgcn_exp2f(fmaf(s[i >> 2][i & 3], scale_log2, -use));
            sum += p[i];
        }
    }
    lsum += sum;
}

// Is any of the wave's accumulators not a number?  (Or its sum not one, which infinities of both signs also give.)
template <int QT, int NT>
__device__ __forceinline__ bool has_nan(const f32x4 (&acc)[QT][NT]) {
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < QT; ++u)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[r] += acc[u][t][r];
    const float all = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    return __any(all != all);
}

// The lane's accumulators of one query tile to a row of floats: accumulator row 4 g + r of tile e of a piece is channel
// base + W (4 g + r) + e.
template <int WMAX, int NT>
__device__ __forceinline__ void frag_store(const f32x4 (&acc)[NT], float* row, int gq) {
    for_pieces<WMAX, NT>([&](auto wd, auto base) {
        constexpr int W = decltype(wd)::value, B0 = decltype(base)::value;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            f32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = acc[B0 / 16 + (4 * i + e) % W][(4 * i + e) / W];
            *reinterpret_cast<f32x4*>(row + B0 + 4 * W * gq + 4 * i) = o;
        }
    });
}

}  // namespace

}  // namespace rr
