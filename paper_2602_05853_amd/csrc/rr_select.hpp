// Adaptive Top-tau selection (Sec. 3.3) of one query-block row by ONE wavefront, shared by the
// estimate kernels.  Input: the row's block-mass fractions in LDS (each row sums to 1).  Output: the
// dense 0/1 row, the ascending list of selected key blocks and their count.
//
// The definition ranks the key blocks by mass (ties: smaller index first) and keeps the shortest prefix
// whose cumulative mass reaches tau.  No sort is needed for that: with g(t) = sum of the fractions >= t,
// the mass of the last kept block is the largest t with g(t) >= tau, and g is a step function whose
// steps sit at the row's own values, so a bisection over the 31 value bits of a non-negative float finds
// it exactly.  Everything above that value is kept, and of the blocks equal to it the first few in index
// order, as many as the cumulative sum still needs.  g is evaluated with one fixed summation order
// (per lane ascending, then a fixed lane tree), which makes it monotone in t in floating point as well.
// The bisection ends as soon as a single value of the row is left between its bounds (that value is the answer:
// g does not change anywhere else between them), about half way on rows of some hundred different masses.
// What bounds it: the chain of these evaluations on few rows, their vector work on many.  Measured (k_select_rows) with the
// sums through the vector ALU, the early end and chunks past the row's end skipped, against all 31 evaluations with sums
// through LDS: 2048 rows of 64 blocks 12.5 -> 7.3 us, 32768 rows of 1024 blocks 124 -> 81 us, 512 rows of 1024 22 -> 17 us.
#pragma once
#include "rr_common.hpp"

namespace rr {

struct SelectRow {
    int nlo, m, Nb;                  // candidates are the key blocks nlo .. m; the row has Nb entries
    float tau;
    bool keep_all;                   // tau = 1, a protected last query block, or a row without an estimate
    int sink_blocks, recent_blocks;  // added after the selection (a union)
    uint8_t* dense;                  // [Nb] or nullptr
    int32_t* list;                   // [Nb]
    int32_t* count;                  // [1]
};

// Sum over the wavefront, the butterfly over lane ^ 1, 2, 4, 8, 16, 32 in that order; every lane gets the result.  Through
// DPP and the lane swaps of the vector ALU: a round trip through LDS per step (ds_bpermute) made this sum most of the
// selection's time.  (Once a quad agrees, its mirror image in the half row is what lane ^ 4 holds, and so on.)
template <int CTRL>
__device__ __forceinline__ float dpp_lane(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_sum_fixed(float v) {
    v += dpp_lane<0xB1>(v);                         // quad_perm [1,0,3,2]
    v += dpp_lane<0x4E>(v);                         // quad_perm [2,3,0,1]
    v += dpp_lane<0x141>(v);                        // row_half_mirror
    v += dpp_lane<0x140>(v);                        // row_mirror
    const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// Row access.  chunk c of a row holds key blocks 64 c .. 64 c + 63, lane l the block 64 c + l; at(c) returns
// this lane's fraction of chunk c, 0 for a block outside the candidates nlo .. m.
//   RowInLds   any row length: the fractions stay in LDS and are read again on every pass
//   RowInRegs  rows of up to 64 * NCH key blocks held in registers (loops over c are unrolled, so the
//              register index is static)
struct RowInLds {
    const float* frac; int nlo, m, lane, c0, c1;
    __device__ __forceinline__ RowInLds(const float* f, int nlo_, int m_, int lane_)
        : frac(f), nlo(nlo_), m(m_), lane(lane_), c0(nlo_ >> 6), c1((m_ >> 6) + 1) {}
    __device__ __forceinline__ float at(int c) const {
        const int n = 64 * c + lane;
        return (n >= nlo && n <= m) ? frac[n] : 0.f;
    }
    template <typename F> __device__ __forceinline__ void for_chunks(F&& f) const {
        for (int c = c0; c < c1; ++c) f(c, at(c));
    }
};
template <int NCH>
struct RowInRegs {
    float v[NCH];
    int c0, c1;                                             // chunks that hold a candidate
    template <typename F> __device__ __forceinline__ void for_chunks(F&& f) const {
        // four chunks to a (wave-uniform) branch: they run side by side, and long rows skip what they do not reach
#pragma unroll
        for (int q = 0; q < NCH; q += 4)
            if (q + 4 > c0 && q < c1) {
#pragma unroll
                for (int c = q; c < q + 4 && c < NCH; ++c) f(c, v[c]);
            }
    }
};

// Called by all 64 lanes of one wavefront.
template <typename Row>
__device__ __forceinline__ void select_row_wave(const Row& row, const SelectRow& r, int lane) {
    const int nlo = r.nlo, m = r.m;
    float tstar = 0.f;                                      // mass of the last kept block
    int ties_kept = 0;                                      // how many blocks equal to it are kept
    bool all = r.keep_all;
    if (!all) {
        int cnt;                                            // fractions >= t of the last evaluation
        auto g = [&](float t) {
            float s = 0.f;
            cnt = 0;
            row.for_chunks([&](int, float f) {
                const bool in = f >= t;
                s += in ? f : 0.f;
                cnt += __popcll(__ballot(in));
            });
            return wave_sum_fixed(s);
        };
        if (!(g(0.f) >= r.tau)) {
            all = true;                                     // the whole row does not reach tau (rounding): keep it
        } else {
            unsigned lo = 0u, hi = 0x7f800001u;             // g(lo) >= tau > g(hi)
            int above_lo = cnt, above_hi = 0;               // fractions >= lo and >= hi
            // fractions below (1 - tau) / (number of candidates) add up to less than 1 - tau: a tight first bound,
            // unless rounding decides otherwise
            const float t0 = (1.f - r.tau) / (float)(m + 1 - nlo);
            if (g(t0) >= r.tau) { lo = __float_as_uint(t0); above_lo = cnt; } else { hi = __float_as_uint(t0); above_hi = cnt; }
            const unsigned one = 0x3f800001u;               // just above 1
            if (hi > one && !(g(__uint_as_float(one)) >= r.tau)) { hi = one; above_hi = cnt; }
            while (hi - lo > 1u && above_lo - above_hi > 1) {
                const unsigned mid = lo + ((hi - lo) >> 1);
                if (g(__uint_as_float(mid)) >= r.tau) { lo = mid; above_lo = cnt; } else { hi = mid; above_hi = cnt; }
            }
            if (hi - lo > 1u) {                             // one fraction in [lo, hi): it is the answer
                const float flo = __uint_as_float(lo), fhi = __uint_as_float(hi);
                float only = 0.f;
                row.for_chunks([&](int, float f) { only += (f >= flo && f < fhi) ? f : 0.f; });
                tstar = wave_sum_fixed(only);               // all other lanes hold 0: exact
            } else {
                tstar = __uint_as_float(lo);                // > 0: the positive entries alone already reach tau
            }
            float above = 0.f;
            int nties = 0;
            row.for_chunks([&](int, float f) {
                above += (f > tstar) ? f : 0.f;
                nties += __popcll(__ballot(f == tstar));
            });
            above = wave_sum_fixed(above);
            float run = above;
            do { run += tstar; ++ties_kept; } while (run < r.tau && ties_kept < nties);
        }
    }
    // flags -> ascending list, count, dense row
    int pos = 0, tie_seen = 0;
    row.for_chunks([&](int c, float f) {
        const int n = 64 * c + lane;
        const bool cand = n >= nlo && n <= m;
        const bool tie = cand && !all && f == tstar;
        const unsigned long long tb = __ballot(tie);
        const int rank = tie_seen + __popcll(tb & ((1ull << lane) - 1ull));
        tie_seen += __popcll(tb);
        const bool sel = cand && (all || f > tstar || (tie && rank < ties_kept) ||
                                  n - nlo < r.sink_blocks || n > m - r.recent_blocks);
        const unsigned long long sb = __ballot(sel);
        if (sel) r.list[pos + __popcll(sb & ((1ull << lane) - 1ull))] = n;
        pos += __popcll(sb);
        if (r.dense && n < r.Nb) r.dense[n] = sel ? 1 : 0;
    });
    if (lane == 0) *r.count = pos;
    // dense entries of the chunks that hold no candidate
    if (r.dense) {
        const int c0 = nlo >> 6, c1 = (m >> 6) + 1;
        for (int c = 0; 64 * c < r.Nb; ++c)
            if ((c < c0 || c >= c1) && 64 * c + lane < r.Nb) r.dense[64 * c + lane] = 0;
    }
}

// The selection of mask row mq of head h of batch bh / Hq (bh = b Hq + h), but for its masses.  has_strides: a row
// without a sampled query (a last block without one complete stride, a decode step that holds none of its block's sampled
// positions) has no estimate and no masses.
__device__ __forceinline__ SelectRow select_row_of(const Geom& g, const EstimateArgs& a, const int32_t* seq_first, long long bh,
                                                   int mq, bool& has_strides) {
    const int Nb = a.Nb, Nbq = g.Lq / a.B;
    const long long row_id = bh * Nbq + mq;
    const int m = mq + (Nb - Nbq);
    int nlo = seq_first ? seq_first[m] : 0;
    nlo = nlo < 0 ? 0 : (nlo > m ? m : nlo);
    const bool last_of_seq = (m == Nb - 1) || (seq_first && seq_first[m + 1] == m + 1);
    const int h = (int)(bh % g.Hq);
    const int off = a.S - 1 - ((a.off_hmul * h + a.off_add) % a.S);
    int r_hi = g.Lr / a.S - m * a.R;                       // strides of the block complete within the length
    r_hi = r_hi > a.R ? a.R : r_hi;
    int r_lo = g.q0 - off - m * a.R * a.S;                 // sampled positions not in front of the step
    r_lo = r_lo <= 0 ? 0 : (r_lo + a.S - 1) / a.S;
    has_strides = r_lo < r_hi;
    SelectRow r;
    r.nlo = nlo; r.m = m; r.Nb = Nb;
    r.tau = a.tau;
    r.keep_all = (a.tau >= 1.0f) || (a.protect_last && last_of_seq);
    r.sink_blocks = a.sink_blocks; r.recent_blocks = a.recent_blocks;
    r.dense = a.dense ? a.dense + row_id * Nb : nullptr;
    r.list = a.row_list + row_id * Nb;
    r.count = a.row_count + row_id;
    return r;
}

// Selection of a row of up to 64 NCH blocks whose masses are in registers, lane l of chunk c holding block 64 c + l and 0 for what
// is no candidate; bm: where its fractions go as well, or nullptr.  Called by all 64 lanes of one wavefront.
template <int NCH>
__device__ __forceinline__ void select_row_of_masses(SelectRow r, RowInRegs<NCH>& row, float* bm, int lane) {
    row.c0 = __builtin_amdgcn_readfirstlane(r.nlo) >> 6;
    row.c1 = (__builtin_amdgcn_readfirstlane(r.m) >> 6) + 1;
    float part = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) part += row.v[c];
    const float total = wave_sum_fixed(part);
    const bool estimated = total > 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        row.v[c] = estimated ? row.v[c] / total : 0.f;
        if (bm && 64 * c + lane < r.Nb) bm[64 * c + lane] = row.v[c];
    }
    r.keep_all = r.keep_all || !estimated;
    select_row_wave(row, r, lane);
}
// The same with the masses in memory (readable for nlo <= n <= m).
template <int NCH>
__device__ __forceinline__ void select_row_in_regs(SelectRow r, bool has_strides, const float* mass, float* bm, int lane) {
    RowInRegs<NCH> row;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int n = 64 * c + lane;
        row.v[c] = (has_strides && n >= r.nlo && n <= r.m) ? mass[n] : 0.f;
    }
    select_row_of_masses(r, row, bm, lane);
}

}  // namespace rr
