// Kernel group (3), generic form: causal block-sparse attention (Sec. 2.1) on the matrix cores for every shape
// the bf16 d = 128, B = 128 kernel does not take: fp32 tensors, any d (a multiple of 8 up to 256), any B up to 128.
//
// Precision.  Nothing is held in fewer than 32 bits: fp32 tensors use the fp32 matrix instructions throughout
// (v_mfma_f32_16x16x4); bf16 tensors form the scores in one bf16 product (exact products, fp32 sums) and split every
// probability exactly into three bf16 terms (3 x 8 of its 24 significant bits) for the product with V.
//
// Work split.  One workgroup per 16 QT queries of a query block; its KW waves walk the row's keys in steps of one or two
// tiles of 16 keys (which may belong to different blocks, so that a block of 48 keys wastes nothing), wave w the
// steps w, w + KW, ..., each with an online softmax of its own, and meet once, in LDS, at the end.  What bounds this
// path is the length of the longest row (the protected last one keeps every block) on the few hundred query blocks
// of such a call, and the traffic between L2 and the compute units (launch_attn_generic chooses QT for both, and 16
// queries to a workgroup for that row).
// Fragments go from global memory (K and V of these shapes stay in L2) straight to registers: with keys split over
// the waves no two of them would share a staged tile, and there is no barrier before the merge.
//
// Measured against the form before it (one workgroup per query block, fp32 vector FMAs on operands staged in LDS, where
// every multiply-add waited for an LDS read): fp32, 1024 tokens, 4 / 2 heads of 64: 576 -> 19 us; fp32, 4096 tokens, 8 / 2
// heads of 128: 5954 -> 175 us (62 TFLOP/s of selected blocks); bf16, 8153 tokens, 16 / 4 heads of 64: 9853 -> 186 us.
//
// Softmax: base 2, the reference is moved only when a wave's sum of a step exceeds 2^8 (all terms of a row share it).
#include "rr_attn_frag.hpp"

namespace rr {

namespace {

__device__ __forceinline__ void store4(float* p, const f32x4& v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ void store4(bf16_t* p, const f32x4& v) {
    const u32x2 o = {f32_to_bf16_bits(v[0]) | (f32_to_bf16_bits(v[1]) << 16),
                     f32_to_bf16_bits(v[2]) | (f32_to_bf16_bits(v[3]) << 16)};
    *reinterpret_cast<u32x2*>(p) = o;
}

constexpr unsigned kMaxGridY = 65535;

template <int NT> constexpr int out_pitch() { return 16 * NT + 4; }

#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) int32_t* scalar_list_t;   // read with scalar loads
#else
typedef const int32_t* scalar_list_t;                                    // the host pass only parses the kernel
#endif

// The 16 QT queries from 16 QT sub on of query block m of head h, by the KW waves of a workgroup.
template <typename T, int NT, int QT, int TL, int KW>
__device__ __forceinline__ void attend(const Geom& g, const AttnArgs& a, float scale_log2, int b, int h, int m, int sub,
                                       float* lds_o, float* lds_ref, float* lds_l) {
    using F = Frag<T, NT, TL>;
    constexpr int kQ = 16 * QT, kPitch = out_pitch<NT>(), kThreads = 64 * KW;
    typedef float (*rows_t)[kQ][kPitch];
    typedef float (*sums_t)[kQ];
    const rows_t s_o = reinterpret_cast<rows_t>(lds_o);
    const sums_t s_ref = reinterpret_cast<sums_t>(lds_ref), s_l = reinterpret_cast<sums_t>(lds_l);

    const int B = a.B, d = g.d, Nb = a.Nb;
    const int t = threadIdx.x, lane = t & 63, x = lane & 15, gq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int Nbq = g.Lq / B;                         // rows of the launch (chunked prefill: the last query blocks)
    const int mq = m - (Nb - Nbq);
    const int kv = h / g.G;
    const long long row_id = ((long long)b * g.Hq + h) * Nbq + mq;
    // row y of the block (position m B + y) is row mq B + y - qoff of Q and O: a step that starts inside its
    // first block has no rows for the first qoff positions of that block
    const long long row0 = (long long)mq * B - g.qoff;
    const T* Q = reinterpret_cast<const T*>(a.Q) + b * g.qsb + h * g.qsh + row0 * g.qsl;
    const T* K = reinterpret_cast<const T*>(a.K) + b * g.ksb + kv * g.ksh;
    const T* V = reinterpret_cast<const T*>(a.V) + b * g.ksb + kv * g.ksh;
    const float NEG_INF = -__builtin_huge_valf();

    // the rows of the block that exist (at least one), and this workgroup's share of them
    const int rows_lo = mq == 0 ? g.qoff : 0;
    const int rows_q = (int)min((long long)B, (long long)(g.Lr - g.q0) - row0);
    const int y0 = kQ * sub;
    if (y0 >= rows_q || y0 + kQ <= rows_lo) return;
    const int y_last = min(y0 + kQ, rows_q) - 1;

    F qf[QT];
#pragma unroll
    for (int u = 0; u < QT; ++u)                      // rows that do not exist: a copy of the nearest real one, not stored
        qf[u].load(Q + (long long)max(min(y0 + 16 * u + x, rows_q - 1), rows_lo) * g.qsl, d, gq);

    // a caller-made list is not trusted with addresses: count held to [0, m+1], entries to [0, m]
    int first = (!a.row_list && a.seq_first) ? a.seq_first[m] : 0;   // dense walk of packed sequences
    first = first < 0 ? 0 : (first > m ? m : first);
    int count = a.row_list ? a.row_count[row_id] : (m + 1 - first);
    count = __builtin_amdgcn_readfirstlane(count < 0 ? 0 : (count > m + 1 ? m + 1 : count));
    const scalar_list_t list = (scalar_list_t)(a.row_list ? a.row_list + row_id * Nb : nullptr);
    auto entry = [&](int i) {                                    // as loaded
        i = i < count ? i : count - 1;
        return list ? list[i] : first + i;
    };
    auto clamp_block = [&](int n) { return n < 0 ? 0 : (n > m ? m : n); };

    // the row's keys: tiles of 16, TB to a block; of a diagonal block at the end of the list only those a query sees
    const int TB = (B + 15) >> 4;
    int tiles = count * TB;
    if (count > 0 && clamp_block(entry(count - 1)) == m) tiles -= TB - 1 - (y_last >> 4);
    const int steps = (tiles + TL - 1) / TL;
    const int step_it = (TL * KW) / TB, step_sub = TL * KW - step_it * TB;   // KW steps on
    int it, ts;                                                  // first tile of the step: entry `it`, tile `ts` of it
    f32x4 acc[QT][NT];
    float ref[QT], lsum[QT];

    // Rows of a tile this lane reads, relative to its first key: row x of K, rows 4 g .. +3 of V.  Keys past the end of
    // the block or of the context are read as a copy of its last one, and masked.
    long long k_off = (long long)x * g.ksl, v_off[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) v_off[r] = (long long)(4 * gq + r) * g.ksl;
    F kf[TL];
    int n[TL], kk[TL], n_next[TL];                               // block and first key inside it; entries of the next step
    auto request = [&]() {                                       // the entries of the step at (it, ts)
#pragma unroll
        for (int tl = 0; tl < TL; ++tl) n_next[tl] = entry(ts + tl >= TB ? it + 1 : it);
    };
    auto advance = [&]() {
        it += step_it;
        ts += step_sub;
        if (ts >= TB) { ts -= TB; ++it; }
    };
    auto last_key = [&](int tl) { return min(B - 1 - kk[tl], g.Lr - 1 - n[tl] * B - kk[tl]); };   // of the tile, if < 15
    auto load_keys = [&]() {                                     // the entries of (it, ts) are in n_next
#pragma unroll
        for (int tl = 0; tl < TL; ++tl) {
            n[tl] = clamp_block(n_next[tl]);
            kk[tl] = 16 * (ts + tl >= TB ? ts + tl - TB : ts + tl);
            const T* base = K + (long long)(n[tl] * B + kk[tl]) * g.ksl;
            const int last = last_key(tl);
            long long off = k_off;
            if (last < 15) off = (long long)min(x, last) * g.ksl;
            kf[tl].load(base + off, d, gq);
        }
    };
    // bf16, whose probabilities are split: all keys a second time where the first met zero times infinity
    constexpr bool kTwoWalks = std::is_same<T, bf16_t>::value;
    auto walk = [&](auto careful) {
    it = (TL * w) / TB;
    ts = TL * w - it * TB;
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        ref[u] = NEG_INF;
        lsum[u] = 0.f;
#pragma unroll
        for (int c = 0; c < NT; ++c) acc[u][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (w < steps) {
        request();
        load_keys();
        advance();
        request();
    }
    for (int st = w; st < steps; st += KW) {
        typename F::V vf;
#pragma unroll
        for (int tl = 0; tl < TL; ++tl) {
            const T* base = V + (long long)(n[tl] * B + kk[tl]) * g.ksl;
            const int last = last_key(tl);
            if (last < 15) {
#pragma unroll
                for (int r = 0; r < 4; ++r) F::load_v(vf, 4 * tl + r, base + (long long)min(4 * gq + r, last) * g.ksl, d, x);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) F::load_v(vf, 4 * tl + r, base + v_off[r], d, x);
            }
        }

        f32x4 s[QT][TL];
#pragma unroll
        for (int u = 0; u < QT; ++u)
#pragma unroll
            for (int tl = 0; tl < TL; ++tl) s[u][tl] = f32x4{0.f, 0.f, 0.f, 0.f};
        F::template qk<QT>(s, kf, qf);
        int last_v[TL];                                          // keys behind it are copies that no row takes
#pragma unroll
        for (int tl = 0; tl < TL; ++tl) {
            const bool diag = n[tl] == m, none = TL * st + tl >= tiles;      // (a tile past the last one)
            last_v[tl] = none ? -1 : last_key(tl);
            if (diag || kk[tl] + 16 > B || none) {
#pragma unroll
                for (int u = 0; u < QT; ++u) {
                    // last key of the lane's four that its query sees: inside the block, and up to the query's own
                    // position in the diagonal one (token causality)
                    int last = diag ? min(B - 1, y0 + 16 * u + x) : B - 1;
                    last = none ? -1 : last - kk[tl] - 4 * gq;
                    f32x4 v = s[u][tl];
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = r > last ? NEG_INF : v[r];
                    s[u][tl] = v;
                }
            }
        }
        // the next step's keys travel during the softmax and the second product, the entries of the one after it
        // through all of the next step
        if (st + KW < steps) {
            load_keys();
            advance();
            request();
        }

        float p[QT][4 * TL];
#pragma unroll
        for (int u = 0; u < QT; ++u)
            frag_softmax<TL, NT>(s[u], scale_log2, ref[u], lsum[u], acc[u], p[u]);
        constexpr bool kCareful = decltype(careful)::value;
        if constexpr (kCareful || !kTwoWalks) {
#pragma unroll
            for (int tl = 0; tl < TL; ++tl)
                if (last_v[tl] < 15) {                           // the same in every lane, and rare
#pragma unroll
                    for (int r = 0; r < 4; ++r) F::drop(vf, 4 * tl + r, 4 * gq + r > last_v[tl]);
                }
        }
        F::template pv<QT, kCareful>(acc, vf, p);
    }
    };
    walk(std::false_type{});
    if constexpr (kTwoWalks)
        if (has_nan(acc)) walk(std::true_type{});

    // ---- the waves' shares, brought to one reference ----
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        float l = lsum[u];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const int q = 16 * u + x;
        if (gq == 0) { s_ref[w][q] = ref[u]; s_l[w][q] = l; }
        frag_store<F::kW, NT>(acc[u], &s_o[w][q][0], gq);
    }
    __syncthreads();
    T* O = reinterpret_cast<T*>(a.O) + b * g.qsb + h * g.qsh + row0 * g.qsl;
    float* lse = a.lse ? a.lse + ((long long)b * g.Hq + h) * (g.Lr - g.q0) + row0 : nullptr;
    for (int idx = t; idx < kQ * 4 * NT; idx += kThreads) {
        const int q = idx / (4 * NT), c = 4 * (idx - q * (4 * NT));
        const int y = y0 + q;
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
        if (y >= rows_lo && y < rows_q) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = l > 0.f ? o[e] / l : 0.f;
            if (c < d) store4(O + (long long)y * g.qsl + c, o);
            if (lse && c == 0) lse[y] = l > 0.f ? top * 0.6931471805599453f + logf(l) : NEG_INF;
        }
    }
}

// QS < QT: the last query block is taken 16 QS queries to a workgroup, by QT / QS times as many (rows of the grid's second axis)
template <typename T, int NT, int QT, int QS, int TL, int KW, int OCC>
__global__ void __launch_bounds__(64 * KW, OCC)
k_attn_generic(Geom g, AttnArgs a, float scale_log2) {
    constexpr int kQ = 16 * QT;
    __shared__ __align__(16) float s_o[KW * kQ * out_pitch<NT>()];
    __shared__ float s_ref[KW * kQ], s_l[KW * kQ];
    const int Nbq = g.Lq / a.B;
    // heaviest rows first (blockIdx.y), heads fastest, and of those the KV head: the XCDs, which take consecutive
    // workgroups in turn, then each keep the keys of few KV heads in L2
    // (more query blocks than the y axis holds: the rest in further turns of the x axis)
    int bx = (int)blockIdx.x, rank = (int)blockIdx.y;
    if (Nbq > (int)kMaxGridY) {
        const int per_row = g.Hq * ((a.B + kQ - 1) / kQ), turn = bx / per_row;
        bx -= turn * per_row;
        if (rank >= Nbq - turn * (int)kMaxGridY) return;
        rank += turn * (int)kMaxGridY;
    }
    int sub = bx / g.Hq;
    const int hx = bx - sub * g.Hq, hl = hx / g.Hkv, kv = hx - hl * g.Hkv;
    const int h = kv * g.G + hl;
    if constexpr (QS < QT) {
        constexpr int kSplit = QT / QS;
        if (rank < kSplit) {
            attend<T, NT, QS, TL, KW>(g, a, scale_log2, blockIdx.z, h, a.Nb - 1, kSplit * sub + rank, s_o, s_ref, s_l);
            return;
        }
        rank -= kSplit - 1;
    }
    attend<T, NT, QT, TL, KW>(g, a, scale_log2, blockIdx.z, h, a.Nb - 1 - rank, sub, s_o, s_ref, s_l);
}

}  // namespace

// Shapes the entry points accept on this path: B (4 d + 19) fp32 words within 150 KB.  A bound of the interface (a caller pads
// or picks B by it); this kernel holds its operands in registers and would take any B up to 128 with any d up to 256.
bool attn_generic_fits(int B, int d) {
    return sizeof(float) * ((size_t)B * (4 * (size_t)d + 19)) <= 150 * 1024;
}

hipError_t launch_attn_generic(const Geom& g, int dtype, const AttnArgs& a, hipStream_t st) {
    const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)g.d));
    auto launch = [&](auto kernel, int queries, int waves, int split) -> hipError_t {
        const unsigned subs = (unsigned)((a.B + queries - 1) / queries);
        const unsigned Nbq = (unsigned)(g.Lq / a.B), turns = (Nbq + kMaxGridY - 1) / kMaxGridY;
        if ((unsigned long long)g.Hq * subs * turns * 64 * waves > 0xFFFFFFFFull) return hipErrorInvalidValue;
        const unsigned ranks = Nbq + (split - 1);
        dim3 grid((unsigned)g.Hq * subs * turns, ranks < kMaxGridY ? ranks : kMaxGridY, g.batch);
        hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), 0, st, g, a, scale_log2);
        return hipGetLastError();
    };
    // Queries per workgroup.  What a workgroup reads of K and V serves its queries only, and the kernel's reads of L2 are
    // its limit on long launches (10-12 TB/s with 16 queries a workgroup); but a row's keys are one workgroup's
    // work, and the longest row (the protected last one keeps every block) should not outlast the rest.  So: few
    // queries where the launch has fewer such workgroups than fill the chip twice, more where it has more.  Measured:
    // fp32, 4096 tokens, 8 heads of 128: 16 queries on four waves 183 us, 32 on eight 176 (dense, 32 heads: 1.80 and
    // 1.51 ms); fp32, 1024 tokens, 4 heads of 64: 19 and 26 us; bf16, 8153 tokens, 16 heads of 64: 32 queries 211 us,
    // 64 queries 182 us (dense 439 and 358 us; wider heads have no registers for 64).
    const long long rows = (long long)g.batch * g.Hq * (g.Lq / a.B);
    auto blocks = [&](int queries) { return rows * ((a.B + queries - 1) / queries); };
    // The last query block 16 queries to a workgroup.  A sparse launch of so few workgroups takes as long as its longest row, and
    // that is the protected last one (attention alone, us; this row alone, the rest alone, both before, now: fp32, 2048 tokens, 8 heads
    // of 128: 89, 58, 91, 60; 4096 tokens, one set of inputs, 166, 134, 168, 145; bf16, 8000 tokens, 8 heads of 64: 114, 90, 121, 89; 4096 tokens,
    // 16 heads 63, 49, 67, 49).  What is gained goes down with the number of workgroups, as other rows come to be nearly as long; the limit
    // lies between the largest that gained (1032) and the smallest that did not (2000).  Estimate and attention, fresh inputs, without / with it, and its workgroups, two runs each:
    //   fp32, 32 queries: 2048 tokens, 8 / 2 heads of 128 (512) 111 / 81; 3000 (752) 147 / 126; 4096 (1024) 192 / 185; 4096, 8 / 2 of 64 (1024) 105 / 99
    //   bf16, 32 or 64 queries: 1500, 8 / 2 of 64, B 32 (376) 42 / 38; 4096, 6 / 3 of 80 (1032) 77 / 69; 4096, 16 / 4 of 64 (1024) 90 / 75;
    //     8000, 8 / 2 of 64 (1000) 152 / 118; 8192, 8 / 2 of 40 (1024) 135 / 104
    // Not where the rest takes longer (2000 workgroups and more: 8153 tokens, 16 heads, attention alone: 126, 141, 146 and with it
    // 146), not for dense calls, whose rows get shorter one by one, and not for further blocks (the last sixteenth of them: 8153
    // tokens 162).
    auto short_last = [&](int queries) {
        return a.row_list && a.B > 16 && blocks(queries) <= 1536 && g.Lq / a.B + queries / 16 <= (int)kMaxGridY;
    };
    auto pick = [&](auto tiles) -> hipError_t {
        constexpr int N = decltype(tiles)::value;
        if constexpr (N > 8) {
            return dtype == RR_BF16 ? launch(k_attn_generic<bf16_t, N, 1, 1, 2, 4, 1>, 16, 4, 1)
                                    : launch(k_attn_generic<float, N, 1, 1, 1, 4, 1>, 16, 4, 1);
        } else {
            if (dtype == RR_BF16) {
                if constexpr (N <= 4)
                    if (a.B > 32 && blocks(64) >= 512)
                        return short_last(64) ? launch(k_attn_generic<bf16_t, N, 4, 1, 2, 4, 2>, 64, 4, 4)
                                              : launch(k_attn_generic<bf16_t, N, 4, 4, 2, 4, 2>, 64, 4, 1);
                return short_last(32) ? launch(k_attn_generic<bf16_t, N, 2, 1, 2, 4, 2>, 32, 4, 2)
                                      : launch(k_attn_generic<bf16_t, N, 2, 2, 2, 4, 2>, 32, 4, 1);
            }
            if (a.B > 16 && blocks(32) >= 512)
                return short_last(32) ? launch(k_attn_generic<float, N, 2, 1, 1, 8, 2>, 32, 8, 2)
                                      : launch(k_attn_generic<float, N, 2, 2, 1, 8, 2>, 32, 8, 1);
            return launch(k_attn_generic<float, N, 1, 1, 1, 8, 2>, 16, 8, 1);
        }
    };
    using std::integral_constant;
    switch ((g.d + 15) / 16) {
#define RR_GENERIC_CASE(N) case N: return pick(integral_constant<int, N>{})
        RR_GENERIC_CASE(1); RR_GENERIC_CASE(2); RR_GENERIC_CASE(3); RR_GENERIC_CASE(4);
        RR_GENERIC_CASE(5); RR_GENERIC_CASE(6); RR_GENERIC_CASE(7); RR_GENERIC_CASE(8);
        RR_GENERIC_CASE(9); RR_GENERIC_CASE(10); RR_GENERIC_CASE(11); RR_GENERIC_CASE(12);
        RR_GENERIC_CASE(13); RR_GENERIC_CASE(14); RR_GENERIC_CASE(15); RR_GENERIC_CASE(16);
#undef RR_GENERIC_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rr
