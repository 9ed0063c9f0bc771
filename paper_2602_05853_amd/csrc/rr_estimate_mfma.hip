// Kernel group (2), MFMA form of the estimation (importance equation, causal stride softmax and block
// mass, Sec. 3.2-3.3) for bf16 tensors with d = 128 and B/S in {4,8,16,32}.
//
// Three forms, by the shape of the call (launch_estimate_mfma), behind one launch that forms the stride sums: contexts of up to
// 1024 key strides in one launch (k_estimate_rows); short steps deep in a longer one in two (k_step_scores, k_step_select);
// everything else, packed sequences and cut diagonal strides of any length among it, in two sweeps (k_stride_mass_mfma) and a
// selection (k_select_rows), which the following describes.
//
// Exactness (of all three).  The stride sums of K are fp32 and must not be rounded to bf16 (that would move
// logits by ~1e-2 and flip far more blocks than the parity margin excuses).  Each fp32 sum is
// instead split exactly into three bf16 terms hi + mid + lo (3 x 8 mantissa bits); Q is bf16
// already, so three bf16 MFMAs with fp32 accumulation reproduce the fp32 products exactly and only
// the accumulation order differs from a plain fp32 dot product.
//
// Work split.  One workgroup per (batch, KV head, group of MB consecutive query blocks).  Its
// "rows" are the sampled queries (Sec. 3.1 positions) of all G query heads of the KV head in those
// blocks, up to 256 of them: this is the GQA sharing -- every staged tile of split stride sums is
// used by all heads of the group.  Wave w owns rows 64w .. 64w+63 as two MFMA column tiles; a
// tile of 32 key strides is the M dimension.  The products are formed transposed (S^T = Ksum Q^T)
// so that a lane owns one sampled query and the softmax statistics of a query are per-lane scalars.
//
// Two sweeps, nothing but the block mass leaves the chip.  The block mass needs every probability
// divided by its query's softmax denominator, which is only known once the query has seen all its
// key strides.  Instead of parking per-(query, key block) partial sums in memory until then, the
// workgroup walks its key tiles twice with the queries held in registers: sweep 1 accumulates each
// query's denominator against a lazily moved reference (no maximum in the common path: the
// reference only moves when a tile's sum of exponentials exceeds 2^10), sweep 2 recomputes the
// scores, forms exp(score - reference) / denominator, sums it over the strides of each key block
// (in-lane and one exchange with lane ^ 32) and over the R sampled queries of a query block (R
// neighbouring lanes, DPP butterfly), and writes one fp32 block mass per (head, query block, key
// block).  The matrix work doubles; the traffic to memory drops by 2 R and the per-row selection
// (k_select_rows) reads R times less.
#include "rr_common.hpp"
#include "rr_select.hpp"

#include <type_traits>

namespace rr {

namespace {

constexpr int kThreads = 256;
constexpr int kTileStrides = 32;
constexpr int kPlaneBytes = kTileStrides * 256;        // 32 strides x 128 bf16
constexpr int kTileBytes = 3 * kPlaneBytes;            // hi, mid, lo
constexpr int kLdsBytes = 2 * kTileBytes;              // double buffered

// ---- stride sums, split into three bf16 planes: Ksp[p][b][kv][j][c], j < LsCap ----
// Eight channels of `nkeys` keys from src on, summed in fp32 in the order of the keys and split.  kAtOnce keys requested at
// once, eight or sixteen (one at a time, a thread's S loads were a chain: 2048 new positions at 128K 11.4 -> 5.0 us, 8K
// tokens, all 8 KV heads 8.3 -> 6.1, 128K 68 -> 63).
template <int kAtOnce>
__device__ __forceinline__ void stride_sum_parts(const Geom& g, const unsigned short* src, int nkeys, u32x4 (&part)[3]) {
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    int s = 0;
    auto take = [&](auto n) {
        constexpr int N = decltype(n)::value;
        for (; s + N <= nkeys; s += N) {
            u32x4 v[N];
#pragma unroll
            for (int u = 0; u < N; ++u) v[u] = *reinterpret_cast<const u32x4*>(src + (s + u) * g.ksl);
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc[2 * i] += __uint_as_float(v[u][i] << 16);
                    acc[2 * i + 1] += __uint_as_float(v[u][i] & 0xFFFF0000u);
                }
        }
    };
    if constexpr (kAtOnce > 8) take(std::integral_constant<int, kAtOnce>{});
    take(std::integral_constant<int, 8>{});
    take(std::integral_constant<int, 1>{});
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x = acc[2 * i], y = acc[2 * i + 1];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const unsigned lo = f32_to_bf16_bits(x), hi = f32_to_bf16_bits(y);
            part[p][i] = lo | (hi << 16);
            x -= __uint_as_float(lo << 16);                // exact: the remainder has fewer bits
            y -= __uint_as_float(hi << 16);
        }
    }
}
__global__ void __launch_bounds__(256)
k_stride_sum_split(Geom g, const unsigned short* __restrict__ K, int S, int Ls, int j0, int LsCap,
                   unsigned short* __restrict__ Ksp) {
    // strides j0 .. Ls-1 (the ones in front are kept from an earlier call); rows of LsCap strides per (batch, KV head)
    const int chunks = g.d / 8, span = Ls - j0;
    const long long total = (long long)g.batch * g.Hkv * span * chunks;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int c = (int)(idx % chunks);
    long long r = idx / chunks;
    const int j = j0 + (int)(r % span);
    r /= span;
    const int kv = (int)(r % g.Hkv);
    const int b = (int)(r / g.Hkv);
    // strides that are not complete within the real length do not exist (Sec. 3.1: floor(L/S) of them): zeros
    u32x4 part[3];
    stride_sum_parts<8>(g, K + b * g.ksb + kv * g.ksh + (long long)j * S * g.ksl + c * 8, (j + 1) * S <= g.Lr ? S : 0, part);
    const long long plane = (long long)g.batch * g.Hkv * LsCap * g.d;
    const long long at = (((long long)(b * g.Hkv + kv) * LsCap + j) * g.d + c * 8);
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4*>(Ksp + p * plane + at) = part[p];
}

// The value lane ^ 32 holds, through the vector ALU (v_permlane32_swap: the upper half of one operand and
// the lower half of the other change places) instead of a round trip through LDS: the tile loop needs it
// five times per query and would otherwise wait for the LDS latency each time.
__device__ __forceinline__ float lane_xor32(float v, bool upper) {
    const unsigned a = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);   // r[0] = (lo, lo), r[1] = (hi, hi)
    return __uint_as_float(upper ? r[0] : r[1]);
}

__device__ __forceinline__ int swz(int row, int chunk) { return row * 256 + ((chunk ^ (row & 15)) << 4); }

struct ScoreArgs {
    const unsigned short* Q;
    const unsigned short* K;        // the keys themselves (diag_token only)
    int diag_token;                 // 1: a query's own stride is cut at the query's position
    const unsigned short* Ksp;      // [3][batch][Hkv][LsCap][128]
    int LsCap;                      // strides the planes are laid out for (>= Ls)
    float* mass;                    // [batch*Hq*Nbq][Nb]: block mass of (row, key block), written for n <= m
    int S, R, Nb, Ls, MB;           // MB query blocks per workgroup
    int off_hmul, off_add;          // sampled offset = S - 1 - ((off_hmul * h + off_add) mod S)
    const int32_t* seq_first;       // packed sequences: first block of the sequence of block m, or nullptr
    float scale_log2;               // log2(e) / (S sqrt(d))
    // Key split: with few workgroups (short contexts, steps) the key tiles of a workgroup's rows are shared out
    // among nsplit workgroups and the two sweeps become two launches.  mode 1: sweep 1 over the own chunk, the
    // softmax state (reference, sum) of every sampled query goes to stats; mode 2: the states of all chunks are
    // combined, then sweep 2 over the own chunk (every key block belongs to exactly one chunk).  mode 0, nsplit
    // 1: both sweeps in one launch.
    float2* stats;                  // [pair][group][nsplit][256]
    int nsplit, mode;
};

// butterfly steps among neighbouring lanes through DPP (no LDS round trip): after xor1 and xor2 all four
// lanes of a quad hold the quad's sum, so "the other quad" / "the other half row" may be reached by mirroring
template <int CTRL>
__device__ __forceinline__ float dpp_get(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// sum over the R lanes l, l^1, .. of an aligned group of R neighbouring lanes; every lane gets the result
template <int R>
__device__ __forceinline__ float group_sum(float v) {
    v += dpp_get<0xB1>(v);                          // quad_perm [1,0,3,2]
    v += dpp_get<0x4E>(v);                          // quad_perm [2,3,0,1]
    if (R >= 8) v += dpp_get<0x141>(v);             // row_half_mirror: lane i <- lane 7 - i
    if (R >= 16) v += dpp_get<0x140>(v);            // row_mirror: lane i <- lane 15 - i
    if (R >= 32) v += __shfl_xor(v, 16);
    return v;
}

constexpr float kLazySum = 1024.0f;                 // a tile's 16-term sum above 2^10 moves the reference

// kExt = false compiles the packed-sequence table and the cut diagonal stride out (the plain method).
// Three workgroups per compute unit (48 KB of LDS and at most 168 registers per lane each): the plain form needs
// 148 registers; the kExt form would take 190 and spills 17-18 of them, which still measured faster than running
// it two to a compute unit.
template <int R, bool kExt>
__global__ void __launch_bounds__(kThreads, 3)
k_stride_mass_mfma(Geom g, ScoreArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int32_t* const seq_first = kExt ? a.seq_first : nullptr;
    const bool diag_token = kExt && a.diag_token != 0;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int l32 = lane & 31, gsel = lane >> 5;
    const int Nbq = g.Lq / (a.R * a.S);                            // query blocks (chunked prefill: the last Nbq)
    const int mfirst = a.Nb - Nbq;
    const int ngroups = (Nbq + a.MB - 1) / a.MB;
    // Launch order: the heaviest groups of ALL (batch, KV head) pairs first.  A group's work grows with its
    // position (the last one walks every key tile, a third of the kernel's duration on its own), so a launch
    // that went KV head by KV head would start half of the heaviest workgroups late and end with a few of
    // them running alone.  Consecutive workgroups go to consecutive XCDs: with the KV head as the fastest
    // index every XCD keeps reading the stride sums of the same few KV heads.
    const int pairs = g.Hkv * g.batch;
    const int chunk = (int)blockIdx.x % a.nsplit, wg = (int)blockIdx.x / a.nsplit;
    const int rank = wg / pairs, pr = wg - rank * pairs;
    const int mg = ngroups - 1 - rank;
    const int b = pr / g.Hkv, kv = pr - b * g.Hkv;
    const int m0 = mfirst + mg * a.MB;
    const int mb = min(a.MB, a.Nb - m0);                           // query blocks in this group
    const int GR = g.G * R;
    const int NR = mb * GR;                                        // rows of this workgroup

    // ---- second launch of a key split: the softmax state of a query over ALL key strides, its states in the chunks
    // brought to one reference.  A lane takes one of the wave's 64 queries and up to 32 chunks at once.  (Both lanes of a
    // query for each of two queries, eight chunks at a time and twice, took 12.7 of the 43 us of such a workgroup for 2048
    // tokens at 128K, 32 chunks; so 3.5.  32K tokens, three chunks, 4.4 -> 2.4.)
    const float NEG_INF = -__builtin_huge_valf();
    float2* const my_stats = a.stats ? a.stats + (((long long)pr * ngroups + mg) * a.nsplit) * 256 : nullptr;
    float state_um = NEG_INF, state_z = 0.f;
    if (a.nsplit > 1 && a.mode == 2) {
        const float2* const sq = my_stats + tid;
        constexpr int kAtOnce = 32;
        float2 part[kAtOnce];
        auto read = [&](int c0) {
#pragma unroll
            for (int u0 = 0; u0 < kAtOnce; u0 += 8) {
                if (c0 + u0 < a.nsplit) {
#pragma unroll
                    for (int u = u0; u < u0 + 8; ++u) part[u] = sq[min(c0 + u, a.nsplit - 1) * 256];
                } else {
#pragma unroll
                    for (int u = u0; u < u0 + 8; ++u) part[u] = make_float2(0.f, 0.f);
                }
            }
        };
        for (int c0 = 0; c0 < a.nsplit; c0 += kAtOnce) {
            read(c0);
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u)                       // (the last chunk again: no new maximum)
                if (part[u].y > 0.f) state_um = fmaxf(state_um, part[u].x);
        }
        for (int c0 = 0; c0 < a.nsplit; c0 += kAtOnce) {
            if (a.nsplit > kAtOnce) read(c0);
#pragma unroll
            for (int u0 = 0; u0 < kAtOnce; u0 += 8) {
                if (c0 + u0 >= a.nsplit) break;
#pragma unroll
                for (int u = u0; u < u0 + 8; ++u)
                    if (c0 + u < a.nsplit && part[u].y > 0.f) state_z += part[u].y * __builtin_amdgcn_exp2f(part[u].x - state_um);
            }
        }
    }

    // ---- this lane's two sampled queries (one per column tile) ----
    bf16x8 qf[2][8];
    int qi_stride[2];                 // query stride index m*R + r, or -1 for a padding row
    int q_lo[2];                      // first key stride the query may see (start of its sequence)
    float* mass_row[2];               // block masses of the query's (head, query block), or nullptr for rows past the group
    int q_m[2];
    float diag_raw[2] = {0.f, 0.f};   // diag_token: Q . (keys of the own stride up to the query), unscaled
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const int q = 64 * wv + 32 * nt + l32;
        const bool in_group = q < NR;
        const int ml = in_group ? q / GR : 0;
        const int rem = in_group ? q - ml * GR : 0;
        const int hl = rem / R, r = rem - hl * R;
        const int h = kv * g.G + hl, m = m0 + ml;
        const long long pos = (long long)(m * R + r) * a.S + (a.S - 1 - ((a.off_hmul * h + a.off_add) % a.S)) - g.q0;   // Sec. 3.1
        // a stride of a partial last block that is not complete within the real length has no sampled query;
        // neither has one whose sampled position lies in front of the step's first query
        const bool valid = in_group && (m * R + r + 1) * a.S <= g.Lr && pos >= 0;
        qi_stride[nt] = valid ? m * R + r : -1;
        q_m[nt] = m;
        {
            int first = (seq_first && in_group) ? seq_first[m] : 0;
            first = first < 0 ? 0 : (first > m ? m : first);      // a malformed table only gives a wrong row
            q_lo[nt] = first * R;
        }
        mass_row[nt] = in_group ? a.mass + (((long long)b * g.Hq + h) * Nbq + (m - mfirst)) * a.Nb : nullptr;
        const unsigned short* qp = a.Q + b * g.qsb + h * g.qsh + pos * g.qsl + 8 * gsel;
#pragma unroll
        for (int kc = 0; kc < 8; ++kc) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (valid) v = *reinterpret_cast<const u32x4*>(qp + 16 * kc);
            qf[nt][kc] = __builtin_bit_cast(bf16x8, v);
        }
        if (diag_token) {
            // this lane holds elements 16 kc + 8 gsel .. +7 of the query; lane ^ 32 holds the others
            const int off = a.S - 1 - ((a.off_hmul * h + a.off_add) % a.S);
            const unsigned short* kp = a.K + b * g.ksb + kv * g.ksh + (long long)(m * R + r) * a.S * g.ksl + 8 * gsel;
            float acc = 0.f;
            if (valid) {
                for (int s = 0; s <= off; ++s) {
#pragma unroll
                    for (int kc = 0; kc < 8; ++kc) {
                        const u32x4 kx = *reinterpret_cast<const u32x4*>(kp + (long long)s * g.ksl + 16 * kc);
                        const u32x4 qx = __builtin_bit_cast(u32x4, qf[nt][kc]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            acc = fmaf(__uint_as_float(qx[e] << 16), __uint_as_float(kx[e] << 16), acc);
                            acc = fmaf(__uint_as_float(qx[e] & 0xFFFF0000u), __uint_as_float(kx[e] & 0xFFFF0000u), acc);
                        }
                    }
                }
            }
            diag_raw[nt] = acc + __shfl_xor(acc, 32);
        }
    }
    // last key stride any row of this wave may see (wave-uniform)
    int wave_last = max(qi_stride[0], qi_stride[1]);
    wave_last = max(wave_last, __shfl_xor(wave_last, 1));
#pragma unroll
    for (int o = 2; o < 64; o <<= 1) wave_last = max(wave_last, __shfl_xor(wave_last, o));
    wave_last = __builtin_amdgcn_readfirstlane(wave_last);
    // first key stride at which some row of this wave needs the causal mask
    int wave_first = qi_stride[0] < 0 ? 0x7fffffff : qi_stride[0];
    wave_first = min(wave_first, qi_stride[1] < 0 ? 0x7fffffff : qi_stride[1]);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) wave_first = min(wave_first, __shfl_xor(wave_first, o));
    wave_first = __builtin_amdgcn_readfirstlane(wave_first);
    // packed sequences: the range of sequence starts among the rows of this wave (both 0 otherwise)
    int lo_min = 0, lo_max = 0;
    if (kExt) {
        lo_min = min(qi_stride[0] < 0 ? 0x7fffffff : q_lo[0], qi_stride[1] < 0 ? 0x7fffffff : q_lo[1]);
        lo_max = max(qi_stride[0] < 0 ? 0 : q_lo[0], qi_stride[1] < 0 ? 0 : q_lo[1]);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            lo_min = min(lo_min, __shfl_xor(lo_min, o));
            lo_max = max(lo_max, __shfl_xor(lo_max, o));
        }
        lo_min = __builtin_amdgcn_readfirstlane(lo_min);
        lo_max = __builtin_amdgcn_readfirstlane(lo_max);
    }

    const int last_stride = (m0 + mb) * R - 1;                     // of the whole workgroup
    const int ntiles = last_stride / kTileStrides + 1;
    int tile0 = 0;                                                 // packed sequences: nothing before block m0's sequence is seen
    if (seq_first) {
        int first = seq_first[m0];
        first = first < 0 ? 0 : (first > m0 ? m0 : first);
        tile0 = first * R / kTileStrides;
    }
    const int span = ntiles - tile0;                               // tiles per sweep
    const long long plane = (long long)g.batch * g.Hkv * a.LsCap * g.d;
    const unsigned short* kbase = a.Ksp + ((long long)(b * g.Hkv + kv) * a.LsCap) * g.d;

    // ---- staging: 3 planes x 32 strides x 256 bytes, copied global -> LDS directly, 1 KB (4 strides) per wave
    // instruction, 6 instructions per wave and tile.  The LDS side of such a copy is lane-contiguous, so the
    // swizzle is applied on the global side: lane (r4, c) of row 4 rg + r4 fetches chunk c ^ (row & 15).
    // Rows past the last stride (last tile only) read the last row: never used unmasked.
    const int r4 = lane >> 4, c16 = lane & 15;
    const int wvu = __builtin_amdgcn_readfirstlane(wv);            // the wave index, known to be the same in every lane
    auto issue_tile = [&](int jt, int buf) {
        const int lim = a.Ls - 1 - jt * kTileStrides;              // last row of the tile that exists (>= 0)
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const int q = wvu + 4 * i;                             // 1 KB piece of the tile: plane q / 8, row group q % 8
            const int p = q >> 3, row = 4 * (q & 7) + r4;
            const unsigned long long srcv = (unsigned long long)(kbase + p * plane + (long long)jt * kTileStrides * g.d);
            // wave-uniform: into scalar registers (readfirstlane yields an int: through unsigned, or the low word
            // is sign-extended over the high one)
            const unsigned src_hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(srcv >> 32));
            const unsigned src_lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)srcv);
            const unsigned short* src =
                reinterpret_cast<const unsigned short*>(((unsigned long long)src_hi << 32) | (unsigned long long)src_lo);
            const unsigned off = 2u * ((unsigned)min(row, lim) * 128u + 8u * (unsigned)(c16 ^ (row & 15)));
            const unsigned dst = (unsigned)(uintptr_t)((__attribute__((address_space(3))) unsigned char*)lds) +
                                 (unsigned)(buf * kTileBytes + p * kPlaneBytes + (q & 7) * 1024);
            asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                         :: "v"(off), "s"(src), "s"(__builtin_amdgcn_readfirstlane(dst)) : "memory");
        }
    };
    auto wait_copies = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };

    // steps t of this workgroup: [0, span) is sweep 1, [span, 2 span) sweep 2; a split workgroup has its chunk
    // of one of them
    int t_begin = 0, t_end = 2 * span;
    if (a.nsplit > 1) {
        const int len = (span + a.nsplit - 1) / a.nsplit;
        const int c_lo = min(span, chunk * len), c_hi = min(span, c_lo + len);
        t_begin = (a.mode == 1 ? 0 : span) + c_lo;
        t_end = (a.mode == 1 ? 0 : span) + c_hi;
        if (a.mode == 2 && t_begin >= t_end) return;               // no key block of these rows is in this chunk
    }
    auto tile_of = [&](int t) { return tile0 + (t >= span ? t - span : t); };

    if (t_begin < t_end) issue_tile(tile_of(t_begin), t_begin & 1);
    // The sampled queries must be complete in their registers before the tile loop: the compiler's waits for
    // ordinary loads count only the loads it knows, and inside the loop they would stall on the tile copies.
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int kc = 0; kc < 8; ++kc) asm volatile("" : "+v"(qf[nt][kc]));
    wait_copies();
    __syncthreads();

    // Softmax state of this lane's share (the strides 8k + 4 gsel .. +3 of every tile) of its two queries, in
    // log2 units: reference U (lazily moved) and sum of 2^(score - U).  Rows that do not exist score 0
    // everywhere (zero query): a finite reference keeps them off the slow path.
    float U[2], Z[2] = {0.f, 0.f}, nbq[2] = {0.f, 0.f}, invZ[2] = {0.f, 0.f};
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) U[nt] = qi_stride[nt] >= 0 ? NEG_INF : 0.f;

    if (a.nsplit > 1 && a.mode == 2) {
        // lanes l and l + 32 of the wave hold the states of its queries in the column tiles 0 and 1
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const float um = __shfl(state_um, 32 * nt + l32), z = __shfl(state_z, 32 * nt + l32);
            nbq[nt] = (um == NEG_INF) ? 0.f : -um;
            invZ[nt] = (qi_stride[nt] >= 0 && z > 0.f) ? 1.0f / z : 0.f;
        }
    }

    // step t: tile tile_of(t) of sweep t / span, in LDS buffer t & 1
    for (int t = t_begin; t < t_end; ++t) {
        const bool sweep2 = t >= span;
        const int jt = tile_of(t);
        const bool more = t + 1 < t_end;
        if (more) issue_tile(tile_of(t + 1), (t + 1) & 1);          // its last readers passed the barrier of step t - 1
        if (t == span && a.nsplit == 1) {
            // between the sweeps: the two lanes of a query hold disjoint strides; combine their states
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const float oU = lane_xor32(U[nt], gsel != 0), oZ = lane_xor32(Z[nt], gsel != 0);
                const float um = fmaxf(U[nt], oU);
                const float use = (um == NEG_INF) ? 0.f : um;
                const float z = Z[nt] * __builtin_amdgcn_exp2f(U[nt] - use) + oZ * __builtin_amdgcn_exp2f(oU - use);
                nbq[nt] = -use;
                invZ[nt] = (qi_stride[nt] >= 0 && z > 0.f) ? 1.0f / z : 0.f;
            }
        }
        const int j0 = jt * kTileStrides;
        if (j0 <= wave_last && j0 + kTileStrides > lo_min) {
            const unsigned char* tile = lds + (t & 1) * kTileBytes;
            f32x16 s[2];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int i = 0; i < 16; ++i) s[nt][i] = 0.f;
#pragma unroll
            for (int kc = 0; kc < 8; ++kc) {
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const bf16x8 kf = *reinterpret_cast<const bf16x8*>(tile + p * kPlaneBytes + swz(l32, 2 * kc + gsel));
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt)
                        s[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[nt][kc], s[nt], 0, 0, 0);
                }
            }
            if (diag_token && j0 + kTileStrides - 1 >= wave_first) {
                // the tile may hold a query's own stride: put the cut score in its place
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (j0 + 8 * (i >> 2) + 4 * gsel + (i & 3) == qi_stride[nt]) s[nt][i] = diag_raw[nt];
            }
            const bool need_mask = j0 + kTileStrides - 1 > wave_first || j0 < lo_max;
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const int iq = qi_stride[nt];
                const int jlo = q_lo[nt];
                if (need_mask) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int j = j0 + 8 * (i >> 2) + 4 * gsel + (i & 3);
                        // causal at stride level (also kills padding rows), and inside the query's own sequence
                        if (j > iq || j < jlo) s[nt][i] = NEG_INF;
                    }
                }
                if (!sweep2) {
                    // ---- sweep 1: denominator against the lazy reference ----
                    const float nb = -U[nt];
                    float sum = 0.f;
#pragma unroll
                    for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(fmaf(s[nt][i], a.scale_log2, nb));
                    // a reference of -inf (nothing seen yet) gives inf or nan and lands here as well
                    const bool move = !(sum <= kLazySum);
                    if (__any(move)) {
                        if (move) {
                            float mx = NEG_INF;
#pragma unroll
                            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[nt][i]);
                            const float top = (mx == NEG_INF) ? NEG_INF : mx * a.scale_log2;
                            const float nu = fmaxf(U[nt], top);
                            const float use = (nu == NEG_INF) ? 0.f : nu;
                            Z[nt] *= __builtin_amdgcn_exp2f(U[nt] - use);      // 0 while the reference is -inf
                            U[nt] = nu;
                            sum = 0.f;
#pragma unroll
                            for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(fmaf(s[nt][i], a.scale_log2, -use));
                        }
                    }
                    Z[nt] += sum;
                } else {
                    // ---- sweep 2: probabilities, summed per key block and over the R queries of a query block ----
                    const float nb = nbq[nt];
                    float e[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) e[i] = __builtin_amdgcn_exp2f(fmaf(s[nt][i], a.scale_log2, nb));
                    constexpr int NBL = (R == 4) ? 4 : kTileStrides / R;       // blocks this lane has a share of
                    constexpr int RPB = 16 / NBL;                               // registers per block
                    const int r = l32 & (R - 1);                                // the query's index inside its block
                    const int m = q_m[nt];
                    const int nlo = jlo / R;
                    float out = 0.f;                                            // the block mass this lane writes
#pragma unroll
                    for (int k = 0; k < NBL; ++k) {
                        float sum = 0.f;
#pragma unroll
                        for (int i = 0; i < RPB; ++i) sum += e[k * RPB + i];
                        // R = 4: a lane holds whole blocks (strides 8k + 4 gsel .. +3 are block 2k + gsel of the
                        // tile); else a block is R/2 consecutive registers here and in lane ^ 32
                        if (R != 4) sum += lane_xor32(sum, gsel != 0);
                        const float tot = group_sum<R>(sum * invZ[nt]);
                        if (r == k) out = tot;
                    }
                    // lane r writes block r of the tile (R = 4: block 2 r + gsel): neighbouring lanes, neighbouring words
                    const int n = (R == 4) ? jt * 8 + 2 * r + gsel : jt * NBL + r;
                    const bool writer = (R == 4) ? true : (gsel == 0 && r < NBL);
                    if (writer && mass_row[nt] && n <= m && n >= nlo) mass_row[nt][n] = out;
                }
            }
        }
        wait_copies();
        __syncthreads();
    }
    if (a.nsplit > 1 && a.mode == 1) {
        // the state of each query over this chunk (the two lanes of a query combined), for the second launch
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const float oU = lane_xor32(U[nt], gsel != 0), oZ = lane_xor32(Z[nt], gsel != 0);
            const float um = fmaxf(U[nt], oU);
            const float use = (um == NEG_INF) ? 0.f : um;
            const float z = Z[nt] * __builtin_amdgcn_exp2f(U[nt] - use) + oZ * __builtin_amdgcn_exp2f(oU - use);
            if (gsel == 0) my_stats[chunk * 256 + 64 * wv + 32 * nt + l32] = make_float2(use, z);
        }
    }
}


// ---- short contexts: scores, softmax, block mass and selection in one launch ----
// Up to 1024 key strides the scores of 64 sampled queries against ALL of them fit the registers of one workgroup: eight
// waves, each TPW tiles of 32 strides (tile w + 8 i) by two column tiles of queries.  The matrix work is then done once
// instead of twice, the softmax needs no second sweep (the waves exchange maxima and sums through LDS), nothing is left for
// another launch, and the workgroup selects its own 64 / R rows, whose masses meet in LDS.  A workgroup takes 64 / R
// consecutive (query block, head) pairs of a KV head, so the heads of a query block share the stride sums it reads; every
// wave has tiles of its own, copied through LDS of its own (see there).
// What bounds it: the chain launch, queries, stride sums, softmax, selection of one row, each waiting for the one before.
// Estimate and attention, us, fragments straight from L2 to registers / through LDS: 32 / 8 heads, 2048 tokens 67.9 / 65.3,
// 8192 231.0 / 223.8, 16384 694.7 / 683.0; 8 / 2, 12000 195.9 / 187.0; 8 tokens of 12000 54.0 / 46.1, 700 of 16000
// 184.5 / 172.7; launches of two workgroups to a compute unit before, which LDS for one now excludes: three prompts of
// 3000, 64 / 8 heads, 293.3 / 294.0, four of 4000, 32 / 8, 324.3 / 323.7.
// A score's exponent is one fma, score scale - round(largest score scale): that rounding is a factor that all strides of a
// query share, and it goes with the sum.  Not where it is itself too large to be an exponent: beyond this reference (log2
// units, rounded to at most 1) the largest score is subtracted first, which leaves its own stride exactly 2^0.  (Without,
// one key of 1e12 made queries drop out of their row, or the row have no estimate.  17 layers and steps with the test for
// it: 0.986 to 1.015 of the time without, twice without 0.992 to 1.008.)
constexpr float kFarReference = 16777216.f;
constexpr int kRowWaves = 8, kRowCols = 64;
constexpr int kQuarterBytes = 3 * kTileStrides * 64;              // 32 channels of a tile's three planes
constexpr int kRowStageBytes = kRowWaves * 2 * kQuarterBytes;
constexpr int kRowTiles = 4 * kRowWaves;                           // the most tiles of key strides it takes
template <int R, int TPW>
__global__ void __launch_bounds__(64 * kRowWaves, 2)
k_estimate_rows(Geom g, ScoreArgs a, EstimateArgs ea) {
    constexpr int P = kRowCols / R;                                // (query block, head) pairs of a workgroup
    constexpr int kMaxNb = kTileStrides * kRowWaves * TPW / R;     // key blocks its tiles cover
    extern __shared__ __align__(16) unsigned char lds_stage[];
    __shared__ float s_red[2][kRowWaves][kRowCols];
    __shared__ float s_mass[P][kMaxNb];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, gsel = lane >> 5;
    const int Nbq = g.Lq / (R * a.S), mfirst = a.Nb - Nbq;
    const int npairs = Nbq * g.G, ngroups = (npairs + P - 1) / P;
    // the last query blocks (the most tiles) first, the KV head fastest, as in k_stride_mass_mfma
    const int kvs = g.Hkv * g.batch;
    const int rank = (int)blockIdx.x / kvs, pr = (int)blockIdx.x - rank * kvs;
    const int p0 = (ngroups - 1 - rank) * P;
    const int b = pr / g.Hkv, kv = pr - b * g.Hkv;
    const int m_last = mfirst + (min(p0 + P, npairs) - 1) / g.G;   // of the workgroup's pairs
    int ntiles = ((m_last + 1) * R - 1) / kTileStrides + 1;
    const int sure = (mfirst + p0 / g.G) * R;                      // every sampled query here sees the strides up to this one

    bf16x8 qf[2][8];
    int qi_stride[2];                 // query stride index m R + r, or -1: no such sampled query
    int q_m[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const int q = 32 * nt + l32, pi = p0 + q / R, r = q & (R - 1);
        const bool in_group = pi < npairs;
        const int ml = in_group ? pi / g.G : 0;
        const int h = kv * g.G + (in_group ? pi - ml * g.G : 0), m = mfirst + ml;
        const long long pos = (long long)(m * R + r) * a.S + (a.S - 1 - ((a.off_hmul * h + a.off_add) % a.S)) - g.q0;   // Sec. 3.1
        const bool valid = in_group && (m * R + r + 1) * a.S <= g.Lr && pos >= 0;
        qi_stride[nt] = valid ? m * R + r : -1;
        q_m[nt] = in_group ? m : -1;
    }
    // Every wave wants the same 64 queries.  The workgroup reads them once, a row of 256 bytes to 16 lanes, into LDS (chunk c of
    // row q in place c ^ (q mod 16)); each of the eight waves for itself read them in touches of 32 bytes of a line, 16 to a row.
    // Estimate and attention, us, before / now: 32 / 8 heads, 1024 tokens 42.4 / 40.5, 2048 65.2 / 62.8, 4096 107.5 / 105.6,
    // 8192 227.7 / 225.9, 16384 689.2 / 685.7; three prompts of 3000, 64 / 8 heads, 297.5 / 290.7; 8 tokens of 12000 46.1 / 46.1.
    {
        u32x4 v[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int q = 8 * w + 4 * t + (lane >> 4), pi = p0 + q / R, r = q & (R - 1);
            const bool in_group = pi < npairs;
            const int ml = in_group ? pi / g.G : 0;
            const int h = kv * g.G + (in_group ? pi - ml * g.G : 0), m = mfirst + ml;
            const long long pos = (long long)(m * R + r) * a.S + (a.S - 1 - ((a.off_hmul * h + a.off_add) % a.S)) - g.q0;
            v[t] = u32x4{0u, 0u, 0u, 0u};
            if (in_group && (m * R + r + 1) * a.S <= g.Lr && pos >= 0)
                v[t] = *reinterpret_cast<const u32x4*>(a.Q + b * g.qsb + h * g.qsh + pos * g.qsl + 8 * ((lane & 15) ^ (q & 15)));
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) *reinterpret_cast<u32x4*>(lds_stage + kRowStageBytes + (8 * w + 4 * t) * 256 + lane * 16) = v[t];
        __syncthreads();
    }
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int kc = 0; kc < 8; ++kc)
            qf[nt][kc] = *reinterpret_cast<const bf16x8*>(lds_stage + kRowStageBytes + swz(32 * nt + l32, 2 * kc + gsel));
    // Every wave holds the same 64 queries.  Where none of them is sampled (most steps of a few tokens complete no stride) no row
    // has an estimate, and nothing is read of the masses: 8 tokens of 31600, S = 32, 32 / 8 heads, estimate and attention
    // 71 us with two sweeps, 84 with the scores here, 51 without; 1 of 16007, S = 16, 47, 58, 39.
    if (!__any(qi_stride[0] >= 0 || qi_stride[1] >= 0)) ntiles = 0;
    const long long plane = (long long)g.batch * g.Hkv * a.LsCap * g.d;
    const unsigned short* kbase = a.Ksp + ((long long)(b * g.Hkv + kv) * a.LsCap) * g.d;
    const float NEG_INF = -__builtin_huge_valf();

    // A wave's tiles, a quarter (32 channels, 3 planes, 6 KB) at a time through LDS of its own, the next quarter on its way
    // meanwhile.
    // The rows of a tile lie 256 bytes apart, so fragments loaded straight to registers took 32 bytes of a line with each
    // of its visits (one a cycle and compute unit): 12 us for the longest workgroup at 8192 tokens; a copy takes 64.  LDS
    // rows of 64 bytes, chunk c of row r in place c ^ (r / 4 mod 4): conflict-free reads.  (Waves read what they copied
    // themselves: no barrier.)
    const unsigned stage = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_stage + (unsigned)(w * 2 * kQuarterBytes);
    const int copy_row = lane >> 2, copy_chunk = (lane & 3) ^ ((lane >> 4) & 3);
    auto issue_quarter = [&](int i, int q) {
        const int j0 = (w + kRowWaves * i) * kTileStrides, lim = a.Ls - 1 - j0;   // rows past the last stride: a copy of it, masked
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const unsigned long long srcv = (unsigned long long)(kbase + p * plane + (long long)j0 * g.d + 32 * q);
            const unsigned src_hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(srcv >> 32));
            const unsigned src_lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)srcv);
            const unsigned short* src =
                reinterpret_cast<const unsigned short*>(((unsigned long long)src_hi << 32) | (unsigned long long)src_lo);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const unsigned off = (unsigned)(min(copy_row + 16 * half, lim) * 256 + copy_chunk * 16);
                const unsigned dst = stage + (unsigned)((q & 1) * kQuarterBytes + p * 2048 + half * 1024);
                asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                             :: "v"(off), "s"(src), "s"(__builtin_amdgcn_readfirstlane(dst)) : "memory");
            }
        }
    };
    typedef __attribute__((address_space(3))) bf16x8 lds_frag_t;
    auto fragment = [&](int q, int p, int k) {
        return *(const lds_frag_t*)(uintptr_t)(stage + (unsigned)((q & 1) * kQuarterBytes + p * 2048 + l32 * 64 + (((2 * k + gsel) ^ ((l32 >> 2) & 3)) << 4)));
    };
    // the queries are complete in their registers here: the waits below count the copies alone
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int kc = 0; kc < 8; ++kc) asm volatile("" : "+v"(qf[nt][kc]));
    f32x16 s[TPW][2];
    float mx[2] = {NEG_INF, NEG_INF};
    if (w < ntiles) issue_quarter(0, 0);
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int jt = w + kRowWaves * i, j0 = jt * kTileStrides;
        if (jt < ntiles) {
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int e = 0; e < 16; ++e) s[i][nt][e] = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // the buffer's fragments of two quarters ago have been read
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (q < 3 || (i + 1 < TPW && jt + kRowWaves < ntiles)) {
                    issue_quarter(q < 3 ? i : i + 1, (q + 1) & 3);
                    asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
                } else {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                }
                bf16x8 kf[2][3];
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int p = 0; p < 3; ++p) kf[k][p] = fragment(q, p, k);
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int p = 0; p < 3; ++p)
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt)
                            s[i][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[k][p], qf[nt][2 * q + k], s[i][nt], 0, 0, 0);
            }
            const bool need_mask = j0 + kTileStrides - 1 > sure;
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const int iq = qi_stride[nt];
                f32x16 v = s[i][nt];
                if (need_mask) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) v[e] = j0 + 8 * (e >> 2) + 4 * gsel + (e & 3) > iq ? NEG_INF : v[e];
                    s[i][nt] = v;
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) mx[nt] = fmaxf(mx[nt], v[e]);
            }
        }
    }
    // the softmax over all key strides: maximum, then sum, of the lane's strides, of the two lanes of a query, of the waves
    float nb[2], sum[2] = {0.f, 0.f}, invZ[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        mx[nt] = fmaxf(mx[nt], lane_xor32(mx[nt], gsel != 0));
        if (gsel == 0) s_red[0][w][32 * nt + l32] = mx[nt];
    }
    __syncthreads();
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        float top = NEG_INF;
#pragma unroll
        for (int i = 0; i < kRowWaves; ++i) top = fmaxf(top, s_red[0][i][32 * nt + l32]);
        nb[nt] = top == NEG_INF ? 0.f : -(top * a.scale_log2);
        const bool is_far = fabsf(nb[nt]) > kFarReference;
        if (__any(is_far)) {
            const float far = is_far ? top : 0.f;                  // (other queries of the wavefront stay what they are)
#pragma unroll
            for (int i = 0; i < TPW; ++i)
                if (w + kRowWaves * i < ntiles) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) s[i][nt][e] -= far;
                }
            nb[nt] = is_far ? 0.f : nb[nt];
        }
    }
#pragma unroll
    for (int i = 0; i < TPW; ++i)
        if (w + kRowWaves * i < ntiles) {
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    s[i][nt][e] = __builtin_amdgcn_exp2f(fmaf(s[i][nt][e], a.scale_log2, nb[nt]));
                    sum[nt] += s[i][nt][e];
                }
        }
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        sum[nt] += lane_xor32(sum[nt], gsel != 0);
        if (gsel == 0) s_red[1][w][32 * nt + l32] = sum[nt];
    }
    __syncthreads();
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        float z = 0.f;
#pragma unroll
        for (int i = 0; i < kRowWaves; ++i) z += s_red[1][i][32 * nt + l32];
        invZ[nt] = (qi_stride[nt] >= 0 && z > 0.f) ? 1.0f / z : 0.f;
    }
    // block masses, as in the second sweep of k_stride_mass_mfma
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int jt = w + kRowWaves * i;
        if (jt < ntiles) {
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                constexpr int NBL = (R == 4) ? 4 : kTileStrides / R;
                constexpr int RPB = 16 / NBL;
                const int r = l32 & (R - 1);
                float out = 0.f;
#pragma unroll
                for (int k = 0; k < NBL; ++k) {
                    float t = 0.f;
#pragma unroll
                    for (int e = 0; e < RPB; ++e) t += s[i][nt][k * RPB + e];
                    if (R != 4) t += lane_xor32(t, gsel != 0);
                    const float tot = group_sum<R>(t * invZ[nt]);
                    if (r == k) out = tot;
                }
                const int n = (R == 4) ? jt * 8 + 2 * r + gsel : jt * NBL + r;
                const bool writer = (R == 4) ? true : (gsel == 0 && r < NBL);
                if (writer && n <= q_m[nt]) s_mass[(32 * nt + l32) / R][n] = out;
            }
        }
    }
    __syncthreads();
    // the rows, one to a wave
    for (int j = w; j < P; j += kRowWaves) {
        const int pi = p0 + j;
        if (pi >= npairs) break;
        const int mq = pi / g.G;
        const long long bh = (long long)b * g.Hq + kv * g.G + (pi - mq * g.G);
        bool has_strides;
        const SelectRow row = select_row_of(g, ea, nullptr, bh, mq, has_strides);
        float* bm = ea.block_mass ? ea.block_mass + (bh * Nbq + mq) * a.Nb : nullptr;
        select_row_in_regs<(kMaxNb + 63) / 64>(row, has_strides, s_mass[j], bm, lane);
    }
}

// ---- short steps: one sweep, then softmax, block masses, selection and row order in one launch ----
// A step of a few tokens has a handful of sampled queries to a KV head, nst strides of each of its G heads, against all key
// strides: a wavefront takes 32 key strides and all queries, 32 at a time, and leaves for each query the sum of 2^(score -
// reference) over each key block and the tile's reference (its largest score).  The second launch, one workgroup to a KV
// head and one wavefront to a row, brings the references together.  What bounds it: the chain of launches and, in each, of
// its loads; 8 tokens behind 64512, 32 / 8 heads: 8 + 10 us, the sums of the new strides among them, where those, the two
// sweeps, the selection and the row order took 5 + 20 + 20 + 9 + 5.
struct StepArgs {
    float* sums;                      // [pair][query][tiles * blocks of a tile]
    float* refs;                      // [pair][query][tiles], log2 units
    int nst, s0;                      // query strides of the step, the first of them
    int tiles;
    int order_shift;
    int j_new;                        // strides from here on have no sums yet: their wavefronts form and keep them
    unsigned short* Ksp;
};
constexpr int kStepWaves = 4;
template <int R>
__global__ void __launch_bounds__(64 * kStepWaves)
k_step_scores(Geom g, ScoreArgs a, StepArgs sa) {
    constexpr int NB = kTileStrides / R;                           // key blocks of a tile
    const int lane = threadIdx.x & 63, l32 = lane & 31, gsel = lane >> 5;
    const int jt = (int)blockIdx.x * kStepWaves + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (jt >= sa.tiles) return;
    const int pr = blockIdx.y, b = pr / g.Hkv, kv = pr - b * g.Hkv, j0 = jt * kTileStrides;
    const long long plane = (long long)g.batch * g.Hkv * a.LsCap * g.d;
    __shared__ u32x4 s_new[2][3][kTileStrides][16];                // up to 32 new strides: two tiles at most
    // (rows that have no sums, or do not exist: one that has)
    const unsigned short* kp = a.Ksp + ((long long)pr * a.LsCap + min(j0 + l32, min(a.Ls, sa.j_new) - 1)) * g.d + 8 * gsel;
    bf16x8 kf[8][3];
#pragma unroll
    for (int kc = 0; kc < 8; ++kc)
#pragma unroll
        for (int p = 0; p < 3; ++p) kf[kc][p] = *reinterpret_cast<const bf16x8*>(kp + p * plane + 16 * kc);
    const int j_end = min(j0 + kTileStrides, a.Ls);
    if (j_end > sa.j_new) {
        // strides without sums: four at a time, 16 lanes to a stride, kept for the calls to come
        for (int r = max(j0, sa.j_new); r < j_end; r += 4) {
            const int j = r + (lane >> 4), c = lane & 15;
            if (j < j_end) {
                u32x4 part[3];
                stride_sum_parts<16>(g, a.K + b * g.ksb + kv * g.ksh + (long long)j * a.S * g.ksl + 8 * c, (j + 1) * a.S <= g.Lr ? a.S : 0, part);
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    *reinterpret_cast<u32x4*>(sa.Ksp + p * plane + ((long long)pr * a.LsCap + j) * g.d + 8 * c) = part[p];
                    s_new[jt & 1][p][j - j0][c] = part[p];
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (j0 + l32 >= sa.j_new && j0 + l32 < j_end) {
#pragma unroll
            for (int kc = 0; kc < 8; ++kc)
#pragma unroll
                for (int p = 0; p < 3; ++p) kf[kc][p] = __builtin_bit_cast(bf16x8, s_new[jt & 1][p][l32][2 * kc + gsel]);
        }
    }
    const float NEG_INF = -__builtin_huge_valf();
    const int nq = g.G * sa.nst;
    for (int q0 = 0; q0 < nq; q0 += 32) {
        const int q = q0 + l32, hl = q / sa.nst, i = sa.s0 + (q - hl * sa.nst);
        const int h = kv * g.G + hl;
        const long long pos = (long long)i * a.S + (a.S - 1 - ((a.off_hmul * h + a.off_add) % a.S)) - g.q0;   // Sec. 3.1
        const bool in = q < nq;
        const int iq = in && pos >= 0 ? i : -1;                    // (every stride of the step is complete)
        const unsigned short* qp = a.Q + b * g.qsb + h * g.qsh + pos * g.qsl + 8 * gsel;
        bf16x8 qf[8];
#pragma unroll
        for (int kc = 0; kc < 8; ++kc) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (iq >= 0) v = *reinterpret_cast<const u32x4*>(qp + 16 * kc);
            qf[kc] = __builtin_bit_cast(bf16x8, v);
        }
        f32x16 s;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
        for (int kc = 0; kc < 8; ++kc)
#pragma unroll
            for (int p = 0; p < 3; ++p) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kc][p], qf[kc], s, 0, 0, 0);
        if (j0 + kTileStrides - 1 > sa.s0 || iq < 0) {
            f32x16 v = s;
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = j0 + 8 * (e >> 2) + 4 * gsel + (e & 3) > iq ? NEG_INF : v[e];
            s = v;
        }
        float mx = NEG_INF;
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[e]);
        mx = fmaxf(mx, lane_xor32(mx, gsel != 0));
        const float top = mx;
        mx *= a.scale_log2;
        float nb = mx == NEG_INF ? 0.f : -mx;
        const bool is_far = fabsf(nb) > kFarReference;
        if (__any(is_far)) {                                       // see there
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] -= is_far ? top : 0.f;
            nb = is_far ? 0.f : nb;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = __builtin_amdgcn_exp2f(fmaf(s[e], a.scale_log2, nb));
        constexpr int NBL = R == 4 ? 4 : NB, RPB = 16 / NBL;
        float* const out = sa.sums + ((long long)pr * nq + q) * (sa.tiles * NB) + jt * NB;
#pragma unroll
        for (int k = 0; k < NBL; ++k) {
            float t = 0.f;
#pragma unroll
            for (int e = 0; e < RPB; ++e) t += s[k * RPB + e];
            if (R != 4) t += lane_xor32(t, gsel != 0);
            if (in && (R == 4 || gsel == 0)) out[R == 4 ? 2 * k + gsel : k] = t;
        }
        if (in && gsel == 0) sa.refs[((long long)pr * nq + q) * sa.tiles + jt] = mx;
    }
}

constexpr int kStepRows = 16;                                      // rows of a KV head
template <int R, int NCH>
__global__ void __launch_bounds__(64 * kStepRows)
k_step_select(Geom g, EstimateArgs ea, StepArgs sa) {
    constexpr int NB = kTileStrides / R;
    __shared__ int s_class[kStepRows];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int kv = blockIdx.x, b = blockIdx.y, pr = b * g.Hkv + kv;
    const int Nbq = g.Lq / ea.B, N = g.G * Nbq, nq = g.G * sa.nst;   // N waves
    const int mr = w / g.G, hl = w - mr * g.G, mq = Nbq - 1 - mr;    // descending block, then head: the order inside a class
    const long long bh = (long long)b * g.Hq + kv * g.G + hl;
    bool has_strides;                                               // (or no query below, no mass, and every block is kept)
    const SelectRow row = select_row_of(g, ea, nullptr, bh, mq, has_strides);
    RowInRegs<NCH> masses;
#pragma unroll
    for (int c = 0; c < NCH; ++c) masses.v[c] = 0.f;
    const int i_lo = max(sa.s0, row.m * R), i_hi = min(sa.s0 + sa.nst, (row.m + 1) * R);
    const float NEG_INF = -__builtin_huge_valf();
    const int off = ea.S - 1 - ((ea.off_hmul * (kv * g.G + hl) + ea.off_add) % ea.S);
    for (int i = i_lo; i < i_hi; ++i) {
        if (i * ea.S + off < g.q0) continue;                        // the sampled position lies in front of the step
        const long long q = (long long)pr * nq + hl * sa.nst + (i - sa.s0);
        const float* const e = sa.sums + q * (sa.tiles * NB);
        const float* const u = sa.refs + q * sa.tiles;
        float ev[NCH], uv[NCH], top = NEG_INF, z = 0.f;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int n = 64 * c + lane;
            const bool in = n <= row.m;
            ev[c] = in ? e[n] : 0.f;
            uv[c] = in ? u[n / NB] : NEG_INF;
            top = fmaxf(top, uv[c]);
        }
        // A query whose scores are no numbers has no largest one, but sums that are no numbers: as in the sweeps they have to reach the
        // row, which then has no estimate and keeps every block.
        top = wave_max(top);
        const float ref = top == NEG_INF ? 0.f : top;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            ev[c] *= __builtin_amdgcn_exp2f(uv[c] - ref);
            z += ev[c];
        }
        z = wave_sum_fixed(z);
        const float inv = z > 0.f ? 1.0f / z : 0.f;
#pragma unroll
        for (int c = 0; c < NCH; ++c) masses.v[c] = fmaf(ev[c], inv, masses.v[c]);
    }
    float* bm = ea.block_mass ? ea.block_mass + (bh * Nbq + mq) * ea.Nb : nullptr;
    select_row_of_masses(row, masses, bm, lane);
    if (!ea.row_order) return;
    // the order k_row_order would give: fewer than 8 G rows are not transposed
    if (ea.queue && pr == 0)
        for (int i = threadIdx.x; i < RR_QUEUE_WORDS; i += 64 * N) ea.queue[i] = 0;
    if (lane == 0) s_class[w] = (ea.Nb - *row.count) >> sa.order_shift;
    __syncthreads();
    if (lane == 0) {
        int rank = 0;
        for (int f = 0; f < N; ++f) rank += s_class[f] < s_class[w] || (s_class[f] == s_class[w] && f < w);
        ea.row_order[(long long)pr * N + rank] = hl * Nbq + mq;
    }
}

}  // namespace

size_t estimate_mfma_ksplit_bytes(const Geom& g, int S) {
    return (size_t)3 * g.batch * g.Hkv * (g.L / S) * g.d * sizeof(unsigned short);
}
// Key split (ScoreArgs::nsplit).  Measured on the 128K workload's generator at 8K .. 128K tokens and on steps:
// a launch of fewer than 1024 workgroups gains from being split into about three times as many (never fewer
// than 768, never more than 1536: beyond that the repeated set-up of a workgroup -- its queries, its first
// tile -- costs more than the idle compute units did), each chunk at least 8 key tiles long.  From 1024
// workgroups on (128K tokens with 8 KV heads) two launches and one are level, and it stays one.
int estimate_mfma_splits(const Geom& g, int S, int B) {
    const int R = B / S, Nbq = g.Lq / B;
    int MB = 256 / (g.G * R);
    if (MB > Nbq) MB = Nbq;
    const long long wgs = (long long)((Nbq + MB - 1) / MB) * g.Hkv * g.batch;
    const int tiles = (g.L / S + kTileStrides - 1) / kTileStrides;
    if (wgs >= 1024) return 1;
    long long target = 3 * wgs;
    target = target < 768 ? 768 : (target > 1536 ? 1536 : target);
    long long P = (target + wgs - 1) / wgs;
    if (P > tiles / 8) P = tiles / 8;
    if (P > 64) P = 64;
    return P < 1 ? 1 : (int)P;
}
size_t estimate_mfma_stats_bytes(const Geom& g, int S, int B) {
    const int P = estimate_mfma_splits(g, S, B);
    if (P <= 1) return 0;
    const int R = B / S, Nbq = g.Lq / B;
    int MB = 256 / (g.G * R);
    if (MB > Nbq) MB = Nbq;
    return (size_t)((Nbq + MB - 1) / MB) * g.Hkv * g.batch * P * 256 * sizeof(float2);
}
size_t estimate_mfma_mass_bytes(const Geom& g, int B) {
    return (size_t)g.batch * g.Hq * (g.Lq / B) * (g.L / B) * sizeof(float);
}
bool estimate_mfma_supported(const Geom& g, int dtype, int S, int B) {
    const int R = B / S;
    return dtype == RR_BF16 && g.d == 128 && (R == 4 || R == 8 || R == 16 || R == 32) && g.G * R <= 256;
}

// Estimate and attention, two sweeps, selection and row order / this form, tau 0.9, us: 32 / 8 heads, 8 tokens of 64512 122 / 89, 1 of
// 98304 141 / 114, 16 of 30000 107 / 75, 40 of 65000 158 / 126; 64 / 8, S = 8, 3 of 90000 212 / 179; 8 / 2, 12 of 20000 83 / 52.  The limit is the
// space: what a workspace of this shape always had for masses and states holds four strides or so of sampled queries, and no
// call may need more than before.
bool estimate_mfma_is_step(const Geom& g, const EstimateArgs& ea) {
    const int S = ea.S, B = ea.B, R = B / S, Nb = g.L / B, Nbq = g.Lq / B;
    const int tiles = (g.L / S + kTileStrides - 1) / kTileStrides;
    const size_t queries = (size_t)g.batch * g.Hq * (g.Lr / S - g.q0 / S);
    const size_t need = queries * (tiles * (kTileStrides / R) + tiles) * sizeof(float);
    return g.q0 > 0 && !ea.seq_first && !ea.diag_token && tiles > kRowTiles && Nb <= 1024 && g.G * Nbq <= kStepRows && Nbq < 8 &&
           g.batch <= 65535 && g.batch * g.Hkv <= 65535 &&
           need <= estimate_mfma_mass_bytes(g, B) + estimate_mfma_stats_bytes(g, S, B);
}

// k_estimate_rows takes the call.
// One launch where its workgroups, which fill a compute unit each and do not overlap one's loads with another's products,
// are less than three to a compute unit.  The whole estimate, us, two sweeps and selection / one launch, with its
// workgroups:
//   32 / 8 heads, S = 16: 8192 tokens (256) 52.4 / 23.1, 12000 (376) 61.0 / 35.9, 16384 (512) 69.3 / 46.9; two prompts of
//     8192 (512) 61.3 / 36.5, four of 5200 (672) 60.8 / 41.7, eight of 2048 (512) 40.7 / 30.6
//   64 / 8: 9000 (568) 62.3 / 43.4, 11000 (688) 71.4 / 50.0; three of 3000 (576) 42.5 / 32.6; 8 / 2, four of 16384 (512)
//     68.7 / 46.8
//   S = 8: 4096, 32 / 8 (256) 50.3 / 22.4, two of 5500 (688) 68.2 / 45.4; S = 32: 16384, 64 / 8 (512) 65.8 / 45.7, 22000
//     (688) 83.0 / 73.0, 32768, 32 / 8 (512) 79.2 / 64.1
// The line was drawn for tiles that went straight to registers, which met the two sweeps there; through LDS they meet
// later: 64 / 8, 16384 (1024) 94.3 / 78.6, S = 8, four of 3000 (768) 61.5 / 39.3, but S = 32, 26000 (816) 88.0 / 89.9, four
// of 9000 (1152) 75.2 / 81.5.
bool short_context(const Geom& g, const EstimateArgs& ea) {
    const int R = ea.B / ea.S, Nbq = g.Lq / ea.B, P = kRowCols / R;
    const int tiles = (g.L / ea.S + kTileStrides - 1) / kTileStrides;
    const long long row_wgs = (long long)((Nbq * g.G + P - 1) / P) * g.Hkv * g.batch;
    return !ea.seq_first && !ea.diag_token && tiles <= kRowTiles && row_wgs <= 700;
}

hipError_t launch_estimate_mfma(const Geom& g, const EstimateArgs& ea, unsigned short* ksplit, int ls_cap, int ls_valid,
                                float* mass, float2* stats, hipStream_t st) {
    const int S = ea.S, B = ea.B, Ls = g.L / S, R = B / S, Nb = g.L / B, Nbq = g.Lq / B;
    if (ls_cap < Ls || ls_valid < 0) return hipErrorInvalidValue;
    const int j0 = ls_valid < Ls ? ls_valid : Ls;
    // A short step's few new strides are left to the wavefronts that score them: a launch of 5 us less.  The bound is on
    // the strides up to the end of the last block, the padding's (which are written as zeros) among them: 32 lie in two
    // tiles at most, which is what s_new holds.  A step that ends early in a block of many strides therefore counts up to a
    // block more than it completes (S = 4: new strides of two blocks are beyond the bound).  Estimate and
    // attention, us: 8 tokens of 64512, 32 / 8 heads, 85.2 -> 81.2, of 30000 47.8 -> 43.4, 1 of 50000 66.8 -> 62.5, 100 of
    // 65000 level.
    const bool step = !short_context(g, ea) && estimate_mfma_is_step(g, ea);
    const bool sums_in_scores = step && j0 > 0 && Ls - j0 <= kTileStrides && g.Lr / S > g.q0 / S;
    if (j0 < Ls && !sums_in_scores) {
        const long long total = (long long)g.batch * g.Hkv * (Ls - j0) * (g.d / 8);
        hipLaunchKernelGGL(k_stride_sum_split, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, g,
                           (const unsigned short*)ea.K, S, Ls, j0, ls_cap, ksplit);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    ScoreArgs a;
    a.Q = (const unsigned short*)ea.Q;
    a.Ksp = ksplit;
    a.LsCap = ls_cap;
    a.mass = mass;
    a.off_hmul = ea.off_hmul;
    a.off_add = ea.off_add;
    a.seq_first = ea.seq_first;
    a.K = (const unsigned short*)ea.K;
    a.diag_token = ea.diag_token;
    a.S = S; a.R = R; a.Nb = Nb; a.Ls = Ls;
    a.MB = 256 / (g.G * R);
    if (a.MB > Nbq) a.MB = Nbq;
    const double sc = 1.0 / ((double)S * sqrt((double)g.d));
    a.scale_log2 = (float)(sc * 1.4426950408889634);
    const bool ext = ea.seq_first != nullptr || ea.diag_token != 0;
    const int tiles = (Ls + kTileStrides - 1) / kTileStrides, P = kRowCols / R;
    const long long row_wgs = (long long)((Nbq * g.G + P - 1) / P) * g.Hkv * g.batch;
    if (short_context(g, ea)) {
        a.nsplit = 1;
        a.mode = 0;
        a.stats = nullptr;
        const dim3 grid((unsigned)row_wgs);
        auto launch = [&](auto kernel) -> hipError_t {
            const hipError_t e = allow_dynamic_lds((const void*)kernel, kRowStageBytes + kRowCols * 256);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(kernel, grid, dim3(64 * kRowWaves), kRowStageBytes + kRowCols * 256, st, g, a, ea);
            return hipGetLastError();
        };
        auto pick = [&](auto r) -> hipError_t {
            constexpr int RV = decltype(r)::value;
            if (tiles <= kRowWaves) return launch(k_estimate_rows<RV, 1>);
            if (tiles <= 2 * kRowWaves) return launch(k_estimate_rows<RV, 2>);
            return launch(k_estimate_rows<RV, 4>);
        };
        switch (R) {
            case 4: return pick(std::integral_constant<int, 4>{});
            case 8: return pick(std::integral_constant<int, 8>{});
            case 16: return pick(std::integral_constant<int, 16>{});
            case 32: return pick(std::integral_constant<int, 32>{});
            default: return hipErrorInvalidValue;
        }
    }
    if (step) {
        a.nsplit = 1;
        a.mode = 0;
        a.stats = nullptr;
        StepArgs sa;
        sa.s0 = g.q0 / S;
        sa.nst = g.Lr / S - sa.s0;
        sa.tiles = tiles;
        sa.sums = mass;
        sa.refs = mass + (size_t)g.batch * g.Hq * sa.nst * (tiles * (kTileStrides / R));
        sa.order_shift = row_order_shift(Nb);
        sa.j_new = sums_in_scores ? j0 : Ls;
        sa.Ksp = ksplit;
        auto launch = [&](auto r) -> hipError_t {
            constexpr int RV = decltype(r)::value;
            if (sa.nst > 0) {
                hipLaunchKernelGGL(k_step_scores<RV>, dim3((unsigned)((tiles + kStepWaves - 1) / kStepWaves), (unsigned)(g.Hkv * g.batch)),
                                   dim3(64 * kStepWaves), 0, st, g, a, sa);
                const hipError_t e = hipGetLastError();
                if (e != hipSuccess) return e;
            }
            const dim3 rows(64 * g.G * Nbq), heads(g.Hkv, g.batch);
            if (Nb <= 256) hipLaunchKernelGGL((k_step_select<RV, 4>), heads, rows, 0, st, g, ea, sa);
            else if (Nb <= 512) hipLaunchKernelGGL((k_step_select<RV, 8>), heads, rows, 0, st, g, ea, sa);
            else hipLaunchKernelGGL((k_step_select<RV, 16>), heads, rows, 0, st, g, ea, sa);
            return hipGetLastError();
        };
        switch (R) {
            case 4: return launch(std::integral_constant<int, 4>{});
            case 8: return launch(std::integral_constant<int, 8>{});
            case 16: return launch(std::integral_constant<int, 16>{});
            case 32: return launch(std::integral_constant<int, 32>{});
            default: return hipErrorInvalidValue;
        }
    }
    const int ngroups = (Nbq + a.MB - 1) / a.MB;
    a.nsplit = stats ? estimate_mfma_splits(g, S, B) : 1;
    a.stats = a.nsplit > 1 ? stats : nullptr;
    dim3 grid((unsigned)ngroups * g.Hkv * g.batch * a.nsplit);
#define RR_LAUNCH_MASS(RV)                                                                          \
    do {                                                                                            \
        if (ext) hipLaunchKernelGGL((k_stride_mass_mfma<RV, true>), grid, dim3(kThreads), kLdsBytes, st, g, a);  \
        else hipLaunchKernelGGL((k_stride_mass_mfma<RV, false>), grid, dim3(kThreads), kLdsBytes, st, g, a);     \
    } while (0)
    // one launch, or (key split) the first sweep and then the second
    for (int pass = (a.nsplit > 1 ? 1 : 0); pass <= (a.nsplit > 1 ? 2 : 0); ++pass) {
        a.mode = pass;
        switch (R) {
            case 4: RR_LAUNCH_MASS(4); break;
            case 8: RR_LAUNCH_MASS(8); break;
            case 16: RR_LAUNCH_MASS(16); break;
            case 32: RR_LAUNCH_MASS(32); break;
            default: return hipErrorInvalidValue;
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
#undef RR_LAUNCH_MASS
    return launch_select_rows(g, ea, mass, st);
}

}  // namespace rr
