// Attention of a short step (one token or a few) against a long context: the decode-stage use of the path (the paper's
// "Future Work"; its experiments decode densely, Sec. 4.1).  bf16, d = 128, B = 128, up to 32 query rows per KV head.
//
// Such a step has G * T query rows per KV head (T tokens, G query heads), too few for a 128-row matrix tile, and its
// cost is reading K and V once.  One workgroup takes a range of key blocks of ONE KV head and serves all G T rows from
// the same keys (the GQA sharing): the rows are the columns of one or two 16 x 16 matrix tiles, the scores one bf16
// product (exact products, fp32 sums), the probabilities split exactly into three bf16 terms for the product with V, so
// that nothing is held in fewer than 32 bits and no row costs vector work per key but its exponential.  Wave w takes keys
// 32 w .. +31 of every block of the range, straight from memory to registers, its next keys requested before the softmax
// of the present ones; each wave runs its own online softmax, the four are merged at the end and the part's normalised
// output and log-sum-exp go to the workspace.  A second kernel merges the parts (the softmax over the selected keys is
// one sum, Sec. 2.1, so parts combine exactly up to rounding).
//
// Sparse steps walk the union of the rows' block lists: a key block is loaded when any row of the KV head
// selected it, and a row skips the blocks it did not select (its scores are masked), so every row still sees
// exactly the blocks of its own list.
//
// What bounds it: the stream of K and V.  Measured, dense, against fp32 vector dot products on the same split (up to 8 rows,
// 16 lanes to a key) and, above 8 rows, a 128-row tile per query head and key range (which reads K and V once per
// query head): 128K tokens, 32 / 8 heads, one token 112 -> 101 us (5.3 TB/s), two 176 -> 105; 64 / 8 heads, one token 175 ->
// 104; 28 / 4 heads, one token 98 -> 56, four 286 -> 78; 16K tokens, one token 27 -> 23; 64K, 8 tokens 143 -> 56.
#include "rr_attn_frag.hpp"
#include "rr_attn_rows.hpp"

#include <algorithm>
#include <type_traits>

namespace rr {

namespace {

constexpr int kDecThreads = 256;
constexpr int kDecMaxRows = 32;         // G * T: two tiles of 16 rows take 254 registers a lane, a third does not fit two waves a SIMD
constexpr int kDecMaxLen = 1024;        // key blocks a part may have
constexpr int kDecMaxParts = 256;
constexpr int kDecBlock = 128;

struct DecodeArgs {
    AttnArgs a;
    int T;              // query positions of the step
    int nblocks;        // key blocks 0 .. nblocks-1 reach the last query
    int len;            // key blocks per part
    int halves;         // 2: a workgroup takes 16 of the rows (QT = 1)
    float scale_log2;   // log2(e) / sqrt(d)
};

// QT: 16-column tiles of query rows, for G T <= 16 or 32; columns beyond G T repeat the last row and are never stored.  (QT = 1
// also takes 32 rows in two workgroups to a part.)
// KW: waves, four to a block of keys and with eight of them two blocks at a time.
template <int QT, int KW>
__global__ void __launch_bounds__(64 * KW, 2)
k_attn_decode(Geom g, DecodeArgs da) {
    constexpr int kThreads = 64 * KW;
    using F = Frag<bf16_t, 8, 2>;
    constexpr int kQ = 16 * QT, kPitch = 132;
    __shared__ __align__(16) float s_o[KW][kQ][kPitch];       // a wave's share: its rows at the end
    static_assert(kPitch >= 128, "a wave's accumulators fit its share");
    __shared__ float s_ref[KW][kQ], s_l[KW][kQ];
    __shared__ unsigned s_sel[kDecMaxLen];                  // which lists hold a block of the range
    __shared__ int s_act[kDecMaxLen];                       // the blocks that any does, as offsets into the range
    __shared__ int s_nact;
    const AttnArgs& a = da.a;
    int part = blockIdx.x, kv = blockIdx.y, b = blockIdx.z, half = 0;
    if (QT == 1 && da.halves == 2) {
        // a grid of one axis: the two workgroups of a part are eight apart, on one XCD, where the second finds the keys in L2
        // (but for up to seven parts at the end)
        const int items = (int)gridDim.x >> 1, full = items & ~7;
        int item = (int)blockIdx.x;
        if (item < 2 * full) {
            half = (item >> 3) & 1;
            item = 8 * (item >> 4) + (item & 7);
        } else {
            item -= full;
            half = item >= items;
            item -= half ? items - full : 0;
        }
        const int pair = item / a.nsplit;
        part = item - pair * a.nsplit;
        b = pair / g.Hkv;
        kv = pair - b * g.Hkv;
    }
    const int tid = threadIdx.x, lane = tid & 63, x = lane & 15, gq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = da.T, R = g.G * T;
    const int Nbq = g.Lq / kDecBlock, m_first = (g.L - g.Lq) / kDecBlock;      // one query block, or two
    const long long nrows = (long long)g.batch * g.Hq * T;
    const float NEG_INF = -__builtin_huge_valf();
    const int lists = g.G * Nbq;                             // at most 32: two query blocks need two tokens

    const bf16_t* Q = reinterpret_cast<const bf16_t*>(a.Q) + b * g.qsb;
    const bf16_t* K = reinterpret_cast<const bf16_t*>(a.K) + b * g.ksb + kv * g.ksh;
    const bf16_t* V = reinterpret_cast<const bf16_t*>(a.V) + b * g.ksb + kv * g.ksh;

    // rows that do not exist repeat the last one and are not stored
    F qf[QT];
    int qpos[QT];
    unsigned mine[QT];                                       // the row's bit in s_sel
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const int rr = min(16 * (half + u) + x, R - 1), hl = rr / T, tk = rr - hl * T;
        qf[u].load(Q + (kv * g.G + hl) * g.qsh + (long long)tk * g.qsl, 128, gq);
        qpos[u] = g.q0 + tk;
        mine[u] = 1u << (hl * Nbq + qpos[u] / kDecBlock - m_first);
    }

    const int n_lo = part * da.len;
    const int n_hi = min(n_lo + da.len, da.nblocks), span = max(n_hi - n_lo, 0);
    // the lists of this workgroup's rows
    unsigned all = lists >= 32 ? 0xFFFFFFFFu : (1u << lists) - 1u;
    if (QT == 1 && da.halves == 2) {
        const int hl_lo = 16 * half / T, hl_hi = min(16 * half + 15, R - 1) / T;
        all &= (unsigned)((1ull << ((hl_hi + 1) * Nbq)) - 1ull) & ~((1u << (hl_lo * Nbq)) - 1u);
    }
    // dense: every block up to a list's own query block (of two query blocks, odd lists are the second's)
    for (int i = tid; i < span; i += kThreads)
        s_sel[i] = a.row_list ? 0u : (n_lo + i <= m_first ? all : (Nbq == 2 ? all & 0xAAAAAAAAu : 0u));
    __syncthreads();
    if (a.row_list) {
        // every list read whole by the workgroup at once (no search: a chain of dependent loads is longer than that);
        // an entry counts where it lies in the range, whatever the list's order
        for (int l = w; l < lists; l += KW) {
            if (!((all >> l) & 1u)) continue;
            const int hl = l / Nbq, mq = l - hl * Nbq;
            const long long rid = ((long long)b * g.Hq + kv * g.G + hl) * Nbq + mq;
            int cn = a.row_count[rid];
            cn = cn < 0 ? 0 : (cn > a.Nb ? a.Nb : cn);
            const int32_t* list = a.row_list + rid * a.Nb;
#pragma unroll 4
            for (int j = lane; j < cn; j += 64) {
                const int e = list[j];
                if (e >= n_lo && e < n_hi && e <= m_first + mq) atomicOr(&s_sel[e - n_lo], 1u << l);
            }
        }
        __syncthreads();
    }
    if (w == 0) {
        int n = 0;
        for (int i0 = 0; i0 < span; i0 += 64) {
            const bool on = i0 + lane < span && s_sel[i0 + lane] != 0u;
            const unsigned long long bal = __ballot(on);
            if (on) s_act[n + __popcll(bal & ((1ull << lane) - 1ull))] = i0 + lane;
            n += __popcll(bal);
        }
        if (lane == 0) s_nact = n;
    }
    __syncthreads();
    const int nact = __builtin_amdgcn_readfirstlane(s_nact);

    f32x4 acc[QT][8];
    float ref[QT], lsum[QT];
    // rows of a tile this lane reads, relative to its first key; keys past the context: a copy of the last, masked
    const long long k_off = (long long)x * g.ksl;
    long long v_off[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) v_off[r] = (long long)(4 * gq + r) * g.ksl;
    F kf[2];
    int key0 = 0;                                            // first key of the wave's 32
    unsigned sel = 0u;
    auto load_keys = [&](int i) {
        const int at = __builtin_amdgcn_readfirstlane(s_act[i]);
        sel = (unsigned)__builtin_amdgcn_readfirstlane((int)s_sel[at]);
        key0 = (n_lo + at) * kDecBlock + 32 * (w & 3);
        const bf16_t* base = K + (long long)key0 * g.ksl;
#pragma unroll
        for (int tl = 0; tl < 2; ++tl) {
            if (key0 + 32 <= g.Lr) kf[tl].load(base + 16 * tl * g.ksl + k_off, 128, gq);
            else kf[tl].load(K + (long long)min(key0 + 16 * tl + x, g.Lr - 1) * g.ksl, 128, gq);
        }
    };
    auto walk = [&](auto careful) {
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        ref[u] = NEG_INF;
        lsum[u] = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[u][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int i0 = w >> 2;
    if (i0 < nact) load_keys(i0);
    for (int i = i0; i < nact; i += KW / 4) {
        typename F::V vf;
        const bf16_t* base = V + (long long)key0 * g.ksl;
        if (key0 + 32 <= g.Lr) {
#pragma unroll
            for (int k = 0; k < 8; ++k) F::load_v(vf, k, base + 16 * (k >> 2) * g.ksl + v_off[k & 3], 128, x);
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                F::load_v(vf, k, V + (long long)min(key0 + 16 * (k >> 2) + 4 * gq + (k & 3), g.Lr - 1) * g.ksl, 128, x);
        }
        f32x4 s[QT][2];
#pragma unroll
        for (int u = 0; u < QT; ++u)
#pragma unroll
            for (int tl = 0; tl < 2; ++tl) s[u][tl] = f32x4{0.f, 0.f, 0.f, 0.f};
        F::template qk<QT>(s, kf, qf);
        const unsigned sel_now = sel;
        const int key_now = key0;
        if (sel != all || key0 + 31 > g.q0) {
#pragma unroll
            for (int u = 0; u < QT; ++u)
#pragma unroll
                for (int tl = 0; tl < 2; ++tl) {
                    // last of the lane's four keys that its row sees: the row selected the block, and token causality
                    const int last = (sel & mine[u]) ? qpos[u] - key0 - 16 * tl - 4 * gq : -1;
                    f32x4 v = s[u][tl];
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = r > last ? NEG_INF : v[r];
                    s[u][tl] = v;
                }
        }
        // travels during the softmax and the second product (the careful walk has no registers for it)
        if (!decltype(careful)::value && i + KW / 4 < nact) load_keys(i + KW / 4);
        float p[QT][8];
#pragma unroll
        for (int u = 0; u < QT; ++u) frag_softmax<2, 8>(s[u], da.scale_log2, ref[u], lsum[u], acc[u], p[u]);
        if constexpr (!decltype(careful)::value) {
            F::template pv<QT, false>(acc, vf, p);
        } else {
            // The values of keys past the context are left out, and a row takes nothing from a block it did not select: its
            // accumulators wait in the wave's share of the merge area meanwhile.
#pragma unroll
            for (int k = 0; k < 8; ++k) F::drop(vf, k, key_now + 16 * (k >> 2) + 4 * gq + (k & 3) >= g.Lr);
            f32x4* const aside = reinterpret_cast<f32x4*>(&s_o[w][0][0]) + lane;
#pragma unroll
            for (int u = 0; u < QT; ++u)
#pragma unroll
                for (int c = 0; c < 8; ++c) aside[64 * (8 * u + c)] = acc[u][c];
            F::template pv<QT, true>(acc, vf, p);
#pragma unroll
            for (int u = 0; u < QT; ++u)
                if ((sel_now & mine[u]) == 0u) {
#pragma unroll
                    for (int c = 0; c < 8; ++c) acc[u][c] = aside[64 * (8 * u + c)];
                }
            if (i + KW / 4 < nact) load_keys(i + KW / 4);
        }
    }
    };
    walk(std::false_type{});
    if (has_nan(acc)) walk(std::true_type{});

    // the waves: the part's normalised output and its natural-log sum of exponentials
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        float l = lsum[u];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (gq == 0) { s_ref[w][16 * u + x] = ref[u]; s_l[w][16 * u + x] = l; }
        frag_store<F::kW, 8>(acc[u], &s_o[w][16 * u + x][0], gq);
    }
    __syncthreads();
    for (int idx = tid; idx < kQ * 32; idx += kThreads) {
        const int q = idx >> 5, c = 4 * (idx & 31), rr = 16 * half + q;
        if (rr >= R) continue;
        float top = NEG_INF;
#pragma unroll
        for (int i = 0; i < KW; ++i) top = fmaxf(top, s_ref[i][q]);
        float l = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KW; ++i) {
            const float f = s_ref[i][q] == NEG_INF ? 0.f : __builtin_amdgcn_exp2f(s_ref[i][q] - top);
            l = fmaf(f, s_l[i][q], l);
            const f32x4 v = *reinterpret_cast<const f32x4*>(&s_o[i][q][c]);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(f, v[e], o[e]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = l > 0.f ? o[e] / l : 0.f;
        const int hl = rr / T, tk = rr - hl * T;
        const long long row = ((long long)b * g.Hq + kv * g.G + hl) * T + tk;
        *reinterpret_cast<f32x4*>(a.part_O + ((long long)part * nrows + row) * 128 + c) = o;
        if (c == 0) a.part_lse[(long long)part * nrows + row] = l > 0.f ? top * 0.6931471805599453f + logf(l) : NEG_INF;
    }
}

// One workgroup per query row: O = sum_p w_p O_p / sum_p w_p with w_p = exp(lse_p - max), rounded once.
__global__ void __launch_bounds__(kDecThreads)
k_attn_decode_combine(Geom g, AttnArgs a, int T) {
    __shared__ float s_w[kDecMaxParts];
    __shared__ float s_red[4];
    __shared__ float s_o[4][128];
    const long long nrows = (long long)g.batch * g.Hq * T;
    const long long row = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int P = a.nsplit;
    const float NEG_INF = -__builtin_huge_valf();
    const float l = tid < P ? a.part_lse[(long long)tid * nrows + row] : NEG_INF;
    float mx = l;
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) mx = fmaxf(mx, __shfl_xor(mx, s));
    if (lane == 0) s_red[wv] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
    const float w = (tid < P && l != NEG_INF) ? expf(l - mx) : 0.f;
    if (tid < kDecMaxParts) s_w[tid] = w;
    __syncthreads();
    // wavefront wv takes the parts p = wv, wv + 4, ..; a lane two channels, up to eight parts requested at once (one at a time, a
    // part of weight zero skipped, their latencies were the kernel: one token of 128K, 64 parts, 8.8 us, so 4.2; 16384 tokens, the
    // whole call 22.1 -> 17.8) and no more than there are (always eight: 4 parts, 16 steps of 2 tokens at 2479, 60 / 4 heads,
    // 21.3 -> 22.5, so 21.1)
    float den = 0.f, o0 = 0.f, o1 = 0.f;
    int p0 = wv;
    auto take = [&](auto n) {
        constexpr int N = decltype(n)::value;
        float2 v[N];
#pragma unroll
        for (int u = 0; u < N; ++u)
            v[u] = *reinterpret_cast<const float2*>(a.part_O + ((long long)min(p0 + 4 * u, P - 1) * nrows + row) * 128 + 2 * lane);
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const float wp = p0 + 4 * u < P ? s_w[p0 + 4 * u] : 0.f;
            if (wp == 0.f) continue;                          // (whatever it holds)
            den += wp;
            o0 = fmaf(wp, v[u].x, o0);
            o1 = fmaf(wp, v[u].y, o1);
        }
        p0 += 4 * N;
    };
    while (p0 + 16 < P) take(std::integral_constant<int, 8>{});
    if (p0 + 4 < P) take(std::integral_constant<int, 4>{});
    if (p0 < P) take(std::integral_constant<int, 1>{});
    __syncthreads();
    if (lane == 0) s_red[wv] = den;
    s_o[wv][2 * lane] = o0;
    s_o[wv][2 * lane + 1] = o1;
    __syncthreads();
    if (wv == 0) {
        den = s_red[0] + s_red[1] + s_red[2] + s_red[3];
        o0 = s_o[0][2 * lane] + s_o[1][2 * lane] + s_o[2][2 * lane] + s_o[3][2 * lane];
        o1 = s_o[0][2 * lane + 1] + s_o[1][2 * lane + 1] + s_o[2][2 * lane + 1] + s_o[3][2 * lane + 1];
        const float inv = den > 0.f ? 1.0f / den : 0.f;
        const long long bh = row / T, t = row - bh * T;
        const int b = (int)(bh / g.Hq), h = (int)(bh - (long long)b * g.Hq);
        unsigned short* O = reinterpret_cast<unsigned short*>(a.O) + b * g.qsb + h * g.qsh + t * g.qsl;
        *reinterpret_cast<unsigned*>(O + 2 * lane) = f32_to_bf16_bits(o0 * inv) | (f32_to_bf16_bits(o1 * inv) << 16);
        if (a.lse && lane == 0) a.lse[row] = den > 0.f ? mx + logf(den) : NEG_INF;
    }
}

}  // namespace

namespace {
// One or two positions of up to 8 rows: no other form serves these, at any depth in the context
bool shortest(const Geom& g) {
    const int T = g.Lr - g.q0;
    return T <= 2 && g.G * T <= 8;
}
size_t part_bytes(const Geom& g) {
    return (size_t)g.batch * g.Hq * (size_t)(g.Lr - g.q0) * (128 + 1) * sizeof(float);
}
// What the launches that the other steps fall back to need of the workspace (0: they do without)
size_t fallback_bytes(const Geom& g, int B) {
    return attn_mfma_plan_len(g, B, nullptr) > 0 ? attn_mfma_plan_bytes(g, B) : attn_mfma_split_bytes(g, B);
}
}  // namespace

// The most parts that pay, 0 when the step is not one of this kernel.  One token: 512 workgroups, two per compute unit (a
// second round of workgroups costs more than longer parts save); steps of more rows, whose parts are wider, 256 (8 tokens
// at 64K, 32 / 8 heads, 512 workgroups 55 us, 256 51; 4 tokens, 28 / 4, 42 and 35).  A part is at least two key blocks
// long.  The shortest steps are taken at any depth; others where all rows lie deep in the context (16 causal blocks or
// more): the limit of the split launch of the 128-row kernel, kept so that the same calls go without a workspace.
int attn_decode_parts(const Geom& g, int B) {
    if (B != kDecBlock || g.d != 128) return 0;
    const int T = g.Lr - g.q0, Nb = g.L / B, Nbq = g.Lq / B;
    if (T < 1) return 0;
    if (g.G * T > kDecMaxRows) return 0;
    if (!shortest(g) && Nb - Nbq + 1 < 16) return 0;
    const int nblocks = (g.Lr - 1) / kDecBlock + 1;
    const long long groups = (long long)g.batch * g.Hkv, target = shortest(g) ? 512 : 256;
    long long P = (target + groups - 1) / groups;
    if (P > (nblocks + 1) / 2) P = (nblocks + 1) / 2;
    if (P > kDecMaxParts) P = kDecMaxParts;
    if (P < 1) P = 1;
    const long long least = (nblocks + kDecMaxLen - 1) / kDecMaxLen;
    if (P < least) P = least;
    if (P > kDecMaxParts) return 0;
    return (int)P;
}

// The bytes a call asks for: all parts of the shortest steps, and for the others no more than the launches that served them
// before ask for, so that the size grows with the step and one workspace serves every step up to the one it was sized for.
// These parts are fewer than fill the chip where the heads of a group are many; eight waves to a workgroup make up for some
// of it, and two workgroups to a part for more.  Dense, us, before the latter: all parts, these, (the split launch): 8
// tokens at 64K, 32 / 8 heads 51, 56, (131); 4 tokens, 28 / 4 heads 35, 45, (177); 64 / 8 heads 51, 89, (239); 32 / 1
// heads, one token, 16 workgroups 30, 50, (218).
size_t attn_decode_bytes(const Geom& g, int B) {
    const int P = attn_decode_parts(g, B);
    if (P < 1) return 0;
    const size_t all = (size_t)P * part_bytes(g), other = fallback_bytes(g, B);
    return shortest(g) || other == 0 ? all : std::min(all, other);
}

int attn_decode_fit(const Geom& g, int B, size_t bytes, bool aligned) {
    const int all = attn_decode_parts(g, B);
    if (all < 1) return 0;
    if (!aligned) return shortest(g) ? -1 : 0;              // (the others check for themselves)
    if (bytes < attn_decode_bytes(g, B) && (shortest(g) || fallback_bytes(g, B) > 0)) return -1;
    const long long fit = std::min<long long>(all, (long long)(bytes / part_bytes(g)));
    const long long nblocks = (g.Lr - 1) / kDecBlock + 1;
    return fit < 1 || (nblocks + fit - 1) / fit > kDecMaxLen ? 0 : (int)fit;
}

// expects 1 <= a.nsplit <= attn_decode_parts(g, a.B), and a.part_O / a.part_lse of that many parts
hipError_t launch_attn_decode(const Geom& g, const AttnArgs& a, hipStream_t st) {
    const int T = g.Lr - g.q0, R = g.G * T;
    if (a.nsplit < 1 || a.nsplit > kDecMaxParts || !a.part_O || !a.part_lse || T < 1 ||
        g.batch > 65535 || g.Hkv > 65535)
        return hipErrorInvalidValue;
    DecodeArgs da;
    da.a = a;
    da.T = T;
    da.nblocks = (g.Lr - 1) / kDecBlock + 1;
    da.len = (da.nblocks + a.nsplit - 1) / a.nsplit;
    da.scale_log2 = (float)(1.4426950408889634 / sqrt((double)g.d));
    if (R > kDecMaxRows || da.len > kDecMaxLen) return hipErrorInvalidValue;
    const DecodeForm form = decode_form(R, (long long)a.nsplit * g.batch * g.Hkv, da.len);
    da.halves = form.halves ? 2 : 1;
    const unsigned parts = (unsigned)a.nsplit;
    const dim3 grid = da.halves == 2 ? dim3(2 * parts * (unsigned)g.Hkv * (unsigned)g.batch) : dim3(parts, (unsigned)g.Hkv, (unsigned)g.batch);
    if (R > 16 && da.halves == 1 && form.eight) hipLaunchKernelGGL((k_attn_decode<2, 8>), grid, dim3(512), 0, st, g, da);
    else if (R > 16 && da.halves == 1) hipLaunchKernelGGL((k_attn_decode<2, 4>), grid, dim3(256), 0, st, g, da);
    else if (form.eight) hipLaunchKernelGGL((k_attn_decode<1, 8>), grid, dim3(512), 0, st, g, da);
    else hipLaunchKernelGGL((k_attn_decode<1, 4>), grid, dim3(256), 0, st, g, da);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long long nrows = (long long)g.batch * g.Hq * T;
    hipLaunchKernelGGL(k_attn_decode_combine, dim3((unsigned)nrows), dim3(kDecThreads), 0, st, g, a, T);
    return hipGetLastError();
}

}  // namespace rr
