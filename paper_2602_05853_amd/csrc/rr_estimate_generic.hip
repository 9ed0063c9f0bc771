// Kernel group (2), generic form: one workgroup per (batch, query head h, query block m) runs
// the whole of Sec. 3.2-3.3 for that row of the block mask without materialising the stride
// score matrix:
//
//   A  scores of the R = B/S sampled queries of block m (Sec. 3.1 positions) against the stride
//      sums of every causal key stride, in chunks; per (sampled query r, key block n) the chunk
//      is reduced at once to a softmax partial (max, sum of exp) -- the "state".
//   B  row maxima and denominators of the causal stride softmax from the state.
//   C  block mass S[m][n] = sum_r state[r][n] rescaled to the row's max / denominator, and its
//      fraction of the row total.
//   D  Top-tau by one wavefront per row (rr_select.hpp: threshold bisection instead of a sort), the last query
//      block keeps every block when protection is on; dense mask row, ascending list and count.
//
// Works for any S | B | L, any d (multiple of 4 for fp32 rows), any group size; fp32 throughout: the scores are formed with
// the fp32 matrix instructions on tiles of 16 key strides x 16 sampled queries.  What bounds it is the score work itself
// and then the selection of the longest rows.  Measured against scores by vector FMAs (a thread per key stride, the
// queries broadcast from LDS), one head per workgroup: 1024 tokens, 4 / 2 heads of 64, fp32 13 -> 12 us; 4096 tokens, 8 / 2
// heads of 128, fp32 37 -> 22 us; 8153 tokens, 16 / 4 heads of 64, bf16 92 -> 33 us.
// The MFMA path covers the benchmark shapes; this one covers everything else and is the
// reference point inside the library.  k_select_rows is the selection stage of the MFMA path: the same
// phase D on block masses that the MFMA kernel left in the workspace.
#include "rr_common.hpp"
#include "rr_estimate_rules.hpp"
#include "rr_select.hpp"

#include <type_traits>

namespace rr {

namespace {

constexpr int kThreads = 256;
constexpr size_t kLdsBudget = 150 * 1024;     // of the 160 KB a workgroup can address

struct EstPlan {
    int CH;          // key strides per chunk (multiple of R)
    int qpitch;      // floats per sampled query in LDS
    int spitch;      // floats per row of scores in LDS
    int frac_pitch;  // floats per row of block masses in LDS
    int state_in_lds;
    int HP;          // query heads of a KV head a workgroup takes
    unsigned off_qs, off_sc, off_state, off_frac, off_scan, off_rows, total;
    size_t budgeted; // what kLdsBudget is compared with: rows of queries rounded up to 8, nothing padded (the
                     // padding is at most 6 KB, which the 160 KB of a compute unit leave room for)
};

// in_lanes: the form that reduces the scores where they are (RF > 0), for HP heads a workgroup
__host__ EstPlan make_plan(const Geom& g, int S, int B, bool in_lanes = false, int HP = 1) {
    EstPlan p;
    const int R = B / S, Nb = g.L / B;
    p.HP = HP;
    int cap = 8192 / R;
    if (cap > 256) cap = 256;
    p.CH = cap / R * R;
    if (p.CH < R) p.CH = R;
    // four floats of padding: the rows that 16 lanes read or write side by side fall on different LDS banks
    p.qpitch = g.d + 4;
    p.spitch = (p.CH + 3) / 4 * 4 + 4;
    int NbP2 = 1;
    while (NbP2 < Nb) NbP2 <<= 1;
    p.frac_pitch = NbP2;
    unsigned o = 0;
    size_t budgeted = 0;
    auto take = [&](size_t bytes, size_t counted) {
        unsigned at = o;
        o += (unsigned)((bytes + 15) / 16 * 16);
        budgeted += (counted + 15) / 16 * 16;
        return at;
    };
    p.off_qs = take((size_t)HP * R * p.qpitch * 4, (size_t)((R + 7) / 8 * 8) * g.d * 4);
    p.off_sc = take(in_lanes ? 0 : (size_t)R * p.spitch * 4, (size_t)R * p.CH * 4);
    p.off_frac = take((size_t)HP * NbP2 * 4, (size_t)NbP2 * 4);
    p.off_scan = take(64, 64);
    p.off_rows = take((size_t)HP * R * 8 + 64, (size_t)R * 8 + 64);
    // the softmax state stays in LDS when it fits beside the rest, else it lives in the workspace
    p.state_in_lds = (budgeted + (size_t)R * Nb * sizeof(float2) <= kLdsBudget) ? 1 : 0;
    const size_t state = p.state_in_lds ? (size_t)R * Nb * 8 : 0;
    p.off_state = take(HP * state, state);
    p.total = o;
    p.budgeted = budgeted;
    return p;
}

// Scores of 32 key strides (two tiles of 16, rows kp0 and kp1 of this lane) against 16 sampled queries (row qrow of this
// lane, in LDS) on the matrix cores, S^T = Ksum Q^T in fp32 (v_mfma_f32_16x16x4); kp0, kp1 and qrow point at channel
// 4 gq.  Lane (x, gq) ends with query x and strides 4 gq .. +3 of each tile.
__device__ __forceinline__ void stride_scores(const float* kp0, const float* kp1, const float* qrow, int d, int gq,
                                              f32x4& acc0, f32x4& acc1) {
    acc0 = f32x4{0.f, 0.f, 0.f, 0.f};
    acc1 = f32x4{0.f, 0.f, 0.f, 0.f};
    const int whole = d & ~15;
    for (int dc = 0; dc < whole; dc += 64) {                          // 64 channels requested at once
        f32x4 k0[4], k1[4], q4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = min(dc + 16 * u, whole - 16);
            k0[u] = *reinterpret_cast<const f32x4*>(kp0 + c);
            k1[u] = *reinterpret_cast<const f32x4*>(kp1 + c);
            q4[u] = *reinterpret_cast<const f32x4*>(qrow + c);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (dc + 16 * u < whole) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(k0[u][e], q4[u][e], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k1[u][e], q4[u][e], acc1, 0, 0, 0);
                }
            }
    }
    if (whole < d) {                                                  // eight more channels: two to a lane
        typedef __attribute__((ext_vector_type(2))) float f32x2;
        const f32x2 k0 = *reinterpret_cast<const f32x2*>(kp0 + whole - 2 * gq);
        const f32x2 k1 = *reinterpret_cast<const f32x2*>(kp1 + whole - 2 * gq);
        const f32x2 q2 = *reinterpret_cast<const f32x2*>(qrow + whole - 2 * gq);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(k0[e], q2[e], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k1[e], q2[e], acc1, 0, 0, 0);
        }
    }
}

// lane ^ 16 and lane ^ 32 through the vector ALU: f(own, other), the same in both lanes
template <typename F>
__device__ __forceinline__ float with_lane16(float v, F&& f) {
    const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return f(__uint_as_float(h[0]), __uint_as_float(h[1]));
}
template <typename F>
__device__ __forceinline__ float with_lane32(float v, F&& f) {
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return f(__uint_as_float(h[0]), __uint_as_float(h[1]));
}

// kExt = false compiles the packed-sequence table and the cut diagonal stride out (the plain method).
// RF: B / S where it is 4, 8, 16 or 32 and kExt is false.  The strides of a key block then sit in whole lanes of a score
// tile and are reduced where they are: nothing goes through LDS but the state, and the waves need no barrier between
// their tiles.  RF = 0: any B / S, the scores of a chunk of strides through LDS.
// W: waves of the workgroup.
template <typename T, bool kExt, int RF, int W>
__global__ void __launch_bounds__(64 * W)
k_estimate_generic(Geom g, EstimateArgs a, EstPlan p, float scale_log2) {
    constexpr int kThreads = 64 * W;
    extern __shared__ __align__(16) unsigned char lds[];
    const int32_t* const seq_first = kExt ? a.seq_first : nullptr;
    const bool diag_token = kExt && a.diag_token != 0;
    float* qs = reinterpret_cast<float*>(lds + p.off_qs);
    float* sc = reinterpret_cast<float*>(lds + p.off_sc);
    float* frac = reinterpret_cast<float*>(lds + p.off_frac);
    float* scanbuf = reinterpret_cast<float*>(lds + p.off_scan);
    float* rowM = reinterpret_cast<float*>(lds + p.off_rows);
    float* rowZ = rowM + p.HP * a.R;                 // reciprocal of the denominator of each sampled query

    const int t = threadIdx.x;
    // Heaviest rows first, heads fastest: a whole launch is resident at once, and with the rows fastest the workgroups a
    // compute unit is dealt (every 256th) were of the same row of several heads, so some units had only the longest.
    const int m = a.Nb - 1 - (int)blockIdx.y;      // the grid covers the Lq/B query blocks
    const int HP = RF > 0 ? p.HP : 1, h0 = (int)blockIdx.x * HP, b = blockIdx.z;   // heads h0 .. h0 + HP - 1
    const int kv = h0 / g.G;
    const int R = a.R, S = a.S, Nb = a.Nb, d = g.d, CH = p.CH;
    const int Ls = g.L / S;
    const int Nbq = g.Lq / a.B;                      // rows of the mask (chunked prefill: < Nb)
    auto row_of = [&](int h) { return ((long long)b * g.Hq + h) * Nbq + (m - (Nb - Nbq)); };
    // packed sequences: row m sees the key blocks nlo .. m of its own sequence; it is that sequence's last
    // query block when the next block starts another one.  A malformed table only gives a wrong row.
    int nlo = seq_first ? seq_first[m] : 0;
    nlo = nlo < 0 ? 0 : (nlo > m ? m : nlo);
    const bool last_of_seq = (m == Nb - 1) || (seq_first && seq_first[m + 1] == m + 1);
    // sampled queries of this block that exist: its strides that are complete within the real length
    // (fewer than R only in a partial last block; none at all: the row has no estimate and keeps every block)
    int Rv = g.Lr / S - m * R;
    Rv = Rv < 0 ? 0 : (Rv > R ? R : Rv);
    // ... and whose sampled position is not in front of the step's first query (a step that starts inside this
    // block): the sampled queries of the row are r = R0 .. Rv - 1
    auto offset_of = [&](int h) { return S - 1 - ((a.off_hmul * h + a.off_add) % S); };
    auto first_of = [&](int h) {
        int r = g.q0 - offset_of(h) - m * R * S;
        r = r <= 0 ? 0 : (r + S - 1) / S;
        return r > R ? R : r;
    };
    const int rows = HP * R;                         // sampled queries of this workgroup: row hh R + r

    float2* state = p.state_in_lds ? reinterpret_cast<float2*>(lds + p.off_state)
                                   : a.state_ws + row_of(h0) * R * Nb;   // (HP = 1)
    const float NEG_INF = -__builtin_huge_valf();

    // ---- sampled queries of this block: position (m*R + r)*S + S-1-(h mod S), Sec. 3.1 ----
    const T* Q = reinterpret_cast<const T*>(a.Q) + b * g.qsb;
    constexpr int VEC = Elem<T>::kVec;
    const int chunks = d / VEC, qp = p.qpitch, sp = p.spitch;
    for (int idx = t; idx < rows * chunks; idx += kThreads) {
        const int q = idx / chunks, c = (idx - q * chunks) * VEC;
        const int h = h0 + q / R, r = q % R;
        float v[VEC];
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = 0.f;
        if (r >= first_of(h) && r < Rv) Elem<T>::load16(Q + h * g.qsh + ((long long)(m * R + r) * S + offset_of(h) - g.q0) * g.qsl + c, v);
#pragma unroll
        for (int i = 0; i < VEC; i += 4) *reinterpret_cast<f32x4*>(qs + q * qp + c + i) = f32x4{v[i], v[i + 1], v[i + 2], v[i + 3]};
    }
    __syncthreads();

    // ---- A: stride scores, reduced per (sampled query, key block) to (max, sum exp) ----
    const float* Ksum = a.Ksum + ((long long)(b * g.Hkv + kv) * Ls) * d;
    const int nstr = (m + 1) * R;
    const int lane = t & 63, wv = t >> 6, x = lane & 15, gq = lane >> 4;
    if constexpr (RF > 0) {
        static_assert(RF == 4 || RF == 8 || RF == 16 || RF == 32, "a block's strides in whole lanes of a tile");
        auto vmax = [](float u, float v) { return fmaxf(u, v); };
        auto vadd = [](float u, float v) { return u + v; };
        for (int j0 = nlo * RF + 32 * wv; j0 < nstr; j0 += 32 * (kThreads / 64)) {
            // strides past the row's last: a copy of it; they are in no block n <= m
            const float* kp0 = Ksum + (long long)min(j0 + x, nstr - 1) * d + 4 * gq;
            const float* kp1 = Ksum + (long long)min(j0 + 16 + x, nstr - 1) * d + 4 * gq;
#pragma unroll
            for (int qt = 0; qt < RF; qt += 16) {
                f32x4 s[2];
                stride_scores(kp0, kp1, qs + min(qt + x, rows - 1) * qp + 4 * gq, d, gq, s[0], s[1]);
                const int q = qt + x, i = m * RF + q % RF;            // row, query stride index
                float mx[2], sum[2];
#pragma unroll
                for (int tl = 0; tl < 2; ++tl) {
                    const int j = j0 + 16 * tl + 4 * gq;
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[tl][e] = j + e <= i ? s[tl][e] * scale_log2 : NEG_INF;   // causal at stride level
                    mx[tl] = fmaxf(fmaxf(s[tl][0], s[tl][1]), fmaxf(s[tl][2], s[tl][3]));
                    if (RF >= 8) mx[tl] = with_lane16(mx[tl], vmax);
                    if (RF >= 16) mx[tl] = with_lane32(mx[tl], vmax);
                }
                if (RF == 32) mx[0] = mx[1] = fmaxf(mx[0], mx[1]);
#pragma unroll
                for (int tl = 0; tl < 2; ++tl) {
                    sum[tl] = 0.f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[tl] += __builtin_amdgcn_exp2f(s[tl][e] - mx[tl]);   // 0 for masked strides
                    if (RF >= 8) sum[tl] = with_lane16(sum[tl], vadd);
                    if (RF >= 16) sum[tl] = with_lane32(sum[tl], vadd);
                }
                if (RF == 32) sum[0] += sum[1];
                constexpr int lanes = RF >= 16 ? 4 : RF / 4;          // values of gq that share a block; the first one writes
#pragma unroll
                for (int tl = 0; tl < (RF == 32 ? 1 : 2); ++tl) {
                    const int n = (j0 + 16 * tl + 4 * gq) / RF;
                    if (q < rows && gq % lanes == 0 && n <= m) state[(long long)q * Nb + n] = make_float2(mx[tl], sum[tl]);
                }
            }
        }
        __syncthreads();
    }
    if constexpr (RF == 0)
    for (int c0 = nlo * R; c0 < nstr; c0 += CH) {
        const int here = min(CH, nstr - c0);                          // strides of this chunk
        for (int j0 = 32 * wv; j0 < here; j0 += 32 * (kThreads / 64)) {
            // strides past the chunk's last: a copy of it, not stored
            const float* kp0 = Ksum + (long long)(c0 + min(j0 + x, here - 1)) * d + 4 * gq;
            const float* kp1 = Ksum + (long long)(c0 + min(j0 + 16 + x, here - 1)) * d + 4 * gq;
            for (int qt = 0; qt < R; qt += 16) {
                f32x4 acc0, acc1;
                stride_scores(kp0, kp1, qs + min(qt + x, R - 1) * qp + 4 * gq, d, gq, acc0, acc1);
                const int r = qt + x, i = m * R + r;                  // query stride index
                if (r < R) {
#pragma unroll
                    for (int tl = 0; tl < 2; ++tl) {
                        const int j = j0 + 16 * tl + 4 * gq;
                        const f32x4 v = tl == 0 ? acc0 : acc1;
                        f32x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = c0 + j + e <= i ? v[e] * scale_log2 : NEG_INF;   // causal at stride level
                        if (j < here) *reinterpret_cast<f32x4*>(sc + r * sp + j) = o;
                    }
                }
            }
        }
        __syncthreads();
        if (diag_token && t >= first_of(h0) && t < Rv) {
            // alternative reading of the diagonal stride: the query at position i*S + off is scored against
            // the keys i*S .. i*S + off of its own stride only (the default sums the whole stride)
            const int i = m * R + t;
            if (i >= c0 && i < c0 + CH) {
                const T* Kd = reinterpret_cast<const T*>(a.K) + b * g.ksb + kv * g.ksh + (long long)i * S * g.ksl;
                const int off = offset_of(h0);
                float acc = 0.f;
                for (int s = 0; s <= off; ++s)
                    for (int c = 0; c < d; ++c) acc = fmaf(qs[t * qp + c], Elem<T>::load1(Kd + (long long)s * g.ksl + c), acc);
                sc[t * sp + (i - c0)] = acc * scale_log2;
            }
        }
        if (diag_token) __syncthreads();
        const int nbc = CH / R;
        for (int pidx = t; pidx < R * nbc; pidx += kThreads) {
            const int nbl = pidx / R, r = pidx - nbl * R;
            const int n = c0 / R + nbl;
            if (n <= m) {
                const float* s = sc + r * sp + nbl * R;
                float mx = NEG_INF;
                for (int jj = 0; jj < R; ++jj) mx = fmaxf(mx, s[jj]);
                float e = 0.f;
                for (int jj = 0; jj < R; ++jj) e += __builtin_amdgcn_exp2f(s[jj] - mx);   // 0 for masked strides
                state[(long long)r * Nb + n] = make_float2(mx, e);
            }
        }
        __syncthreads();
    }

    // ---- B: row maximum and denominator of the causal stride softmax ----
    {
        for (int r = wv; r < rows; r += kThreads / 64) {
            float mx = NEG_INF;
            for (int n = nlo + lane; n <= m; n += 64) mx = fmaxf(mx, state[(long long)r * Nb + n].x);
            mx = wave_max(mx);
            float z = 0.f;
            for (int n = nlo + lane; n <= m; n += 64) {
                const float2 v = state[(long long)r * Nb + n];
                z += v.y * __builtin_amdgcn_exp2f(v.x - mx);
            }
            z = wave_sum_fixed(z);
            if (lane == 0) { rowM[r] = mx; rowZ[r] = 1.0f / z; }
        }
    }
    __syncthreads();

    // ---- C: block mass of every head's row ----
    const int fp = p.frac_pitch;
    for (int hh = 0; hh < HP; ++hh) {
        const int r_lo = first_of(h0 + hh);
        const float2* sh = state + (long long)hh * R * Nb;
        float part = 0.f;
        for (int n = nlo + t; n <= m; n += kThreads) {
            float mass = 0.f;
            for (int r = r_lo; r < Rv; ++r) {
                const float2 v = sh[(long long)r * Nb + n];
                mass += v.y * __builtin_amdgcn_exp2f(v.x - rowM[hh * R + r]) * rowZ[hh * R + r];
            }
            frac[hh * fp + n] = mass;
            part += mass;
        }
        part = wave_sum_fixed(part);
        if (lane == 0 && (W == 4 || wv < 4)) scanbuf[4 * hh + wv] = part;     // (W > 4: up to 256 blocks, nothing behind them)
    }
    __syncthreads();

    // ---- D: fractions of the row total, Top-tau, union with sink / recent blocks, outputs: one wavefront per head ----
    if (wv < HP) {
        const int h = h0 + wv;
        const long long row_id = row_of(h);
        const bool sampled = Rv > first_of(h);
        const float total = scanbuf[4 * wv] + scanbuf[4 * wv + 1] + scanbuf[4 * wv + 2] + scanbuf[4 * wv + 3];
        float* const mine = frac + wv * fp;
        for (int n = nlo + lane; n <= m; n += 64) mine[n] = sampled ? mine[n] / total : 0.f;   // read back by the same lane
        if (a.block_mass) {
            float* bm = a.block_mass + row_id * Nb;
            for (int n = lane; n < nlo; n += 64) bm[n] = 0.f;
            for (int n = nlo + lane; n < Nb; n += 64) bm[n] = n <= m ? mine[n] : 0.f;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        SelectRow r;
        r.nlo = nlo; r.m = m; r.Nb = Nb;
        r.tau = a.tau;
        r.keep_all = (a.tau >= 1.0f) || (a.protect_last && last_of_seq) || !sampled;
        r.sink_blocks = a.sink_blocks; r.recent_blocks = a.recent_blocks;
        r.dense = a.dense ? a.dense + row_id * Nb : nullptr;
        r.list = a.row_list + row_id * Nb;
        r.count = a.row_count + row_id;
        if (Nb <= 256) {                               // in registers: the bisection reads the row some twenty times
            RowInRegs<4> row;
            row.c0 = nlo >> 6;
            row.c1 = (m >> 6) + 1;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int n = 64 * c + lane;
                row.v[c] = (n >= nlo && n <= m) ? mine[n] : 0.f;
            }
            select_row_wave(row, r, lane);
        } else {
            select_row_wave(RowInLds(mine, nlo, m, lane), r, lane);
        }
    }
}

// Selection stage of the MFMA path: one wavefront per mask row.  mass[row][n] holds the block masses
// (Sec. 3.3 block-importance equation: stride-softmax probabilities summed over the R x R strides of a
// block pair) for nlo <= n <= m; the row total normalises them, then phase D as above.
// NCH > 0: rows of up to 64 * NCH key blocks, held in registers; NCH = 0: any length, through LDS.
template <bool kExt, int NCH>
__global__ void __launch_bounds__(kThreads)
k_select_rows(Geom g, EstimateArgs a, const float* __restrict__ mass, long long rows) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int32_t* const seq_first = kExt ? a.seq_first : nullptr;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int Nb = a.Nb, Nbq = g.Lq / a.B;
    // heaviest rows (largest m) first; the four rows of a workgroup are neighbours in m
    const long long slot = (long long)blockIdx.x * (kThreads / 64) + w;
    if (slot >= rows) return;
    const int mq = Nbq - 1 - (int)(slot % Nbq);
    const long long bh = slot / Nbq;
    const long long row_id = bh * Nbq + mq;
    bool has_strides;
    SelectRow r = select_row_of(g, a, seq_first, bh, mq, has_strides);
    const int nlo = r.nlo, m = r.m;
    const float* src = mass + row_id * Nb;
    float* bm = a.block_mass ? a.block_mass + row_id * Nb : nullptr;
    if (NCH > 0) {
        select_row_in_regs<(NCH > 0 ? NCH : 1)>(r, has_strides, src, bm, lane);
    } else {
        float* frac = reinterpret_cast<float*>(lds) + (size_t)w * ((Nb + 63) / 64 * 64);
        float part = 0.f;
        for (int n = nlo + lane; n <= m; n += 64) {
            const float v = has_strides ? src[n] : 0.f;
            frac[n] = v;
            part += v;
        }
        const float total = wave_sum_fixed(part);
        const bool estimated = total > 0.f;
        for (int n = nlo + lane; n <= m; n += 64) frac[n] = estimated ? frac[n] / total : 0.f;
        if (bm)
            for (int n = lane; n < Nb; n += 64) bm[n] = (n >= nlo && n <= m) ? frac[n] : 0.f;
        r.keep_all = r.keep_all || !estimated;
        select_row_wave(RowInLds(frac, nlo, m, lane), r, lane);
    }
}

}  // namespace

bool estimate_generic_fits(const Geom& g, int S, int B) {
    return make_plan(g, S, B).budgeted <= kLdsBudget;
}

size_t estimate_generic_state_bytes(const Geom& g, int S, int B) {
    const EstPlan p = make_plan(g, S, B);
    if (p.state_in_lds) return 0;
    return (size_t)g.batch * g.Hq * (g.Lq / B) * (B / S) * (g.L / B) * sizeof(float2);
}

hipError_t launch_estimate_generic(const Geom& g, int dtype, const EstimateArgs& a, hipStream_t st) {
    const bool ext = a.seq_first != nullptr || a.diag_token != 0;
    const bool in_lanes = !ext && (a.R == 4 || a.R == 8 || a.R == 16 || a.R == 32);
    // A score tile has 16 columns: heads of the KV head share it as long as their sampled queries fit and the state of
    // all of them leaves room for two workgroups on a compute unit (8153 tokens, 16 / 4 heads, 8 queries a block: one head
    // 54 us, two 33 us)
    EstPlan p = make_plan(g, a.S, a.B, in_lanes);
    if (in_lanes && p.state_in_lds)
        for (int hp = 4; hp >= 2; hp >>= 1) {
            const EstPlan q = make_plan(g, a.S, a.B, true, hp);
            if (a.R * hp <= 16 && g.G % hp == 0 && q.total <= 80 * 1024) { p = q; break; }
        }
    const float scale_log2 = (float)(1.4426950408889634 / ((double)a.S * sqrt((double)g.d)));
    dim3 grid(g.Hq / p.HP, g.Lq / a.B, g.batch);
    auto launch = [&](auto kernel, int waves) -> hipError_t {
        hipError_t e = allow_dynamic_lds((const void*)kernel, p.total);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), p.total, st, g, a, p, scale_log2);
        return hipGetLastError();
    };
    const bool eight = eight_waves_pay((long long)grid.x * grid.y * grid.z, g.batch, a.Nb, a.R, p.HP, g.d, p.total);
    auto launch_waves = [&](auto type, auto r) -> hipError_t {
        using T = decltype(type);
        constexpr int RF = decltype(r)::value;
        return eight ? launch(k_estimate_generic<T, false, RF, 8>, 8) : launch(k_estimate_generic<T, false, RF, 4>, 4);
    };
    auto launch_type = [&](auto type) -> hipError_t {
        using T = decltype(type);
        using std::integral_constant;
        if (ext) return launch(k_estimate_generic<T, true, 0, 4>, 4);
        switch (a.R) {
            case 4: return launch_waves(T{}, integral_constant<int, 4>{});
            case 8: return launch_waves(T{}, integral_constant<int, 8>{});
            case 16: return launch_waves(T{}, integral_constant<int, 16>{});
            case 32: return launch_waves(T{}, integral_constant<int, 32>{});
            default: return launch(k_estimate_generic<T, false, 0, 4>, 4);
        }
    };
    return dtype == RR_BF16 ? launch_type(bf16_t{}) : launch_type(float{});
}

hipError_t launch_select_rows(const Geom& g, const EstimateArgs& a, const float* mass, hipStream_t st) {
    const long long rows = (long long)g.batch * g.Hq * (g.Lq / a.B);
    const int nch = a.Nb <= 256 ? 4 : (a.Nb <= 512 ? 8 : (a.Nb <= 1024 ? 16 : 0));
    const unsigned lds_bytes = nch ? 0u : (unsigned)((kThreads / 64) * ((a.Nb + 63) / 64 * 64) * sizeof(float));
    const dim3 grid((unsigned)((rows + kThreads / 64 - 1) / (kThreads / 64)));
    auto launch = [&](auto kernel) -> hipError_t {
        if (lds_bytes > 48 * 1024) {
            hipError_t e = allow_dynamic_lds((const void*)kernel, lds_bytes);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, grid, dim3(kThreads), lds_bytes, st, g, a, mass, rows);
        return hipGetLastError();
    };
    const bool ext = a.seq_first != nullptr;
    switch (nch) {
        case 4: return ext ? launch(k_select_rows<true, 4>) : launch(k_select_rows<false, 4>);
        case 8: return ext ? launch(k_select_rows<true, 8>) : launch(k_select_rows<false, 8>);
        case 16: return ext ? launch(k_select_rows<true, 16>) : launch(k_select_rows<false, 16>);
        default: return ext ? launch(k_select_rows<true, 0>) : launch(k_select_rows<false, 0>);
    }
}

}  // namespace rr
