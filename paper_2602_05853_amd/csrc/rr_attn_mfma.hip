// Kernel group (3), MFMA form: causal block-sparse flash attention (Sec. 2.1) for bf16 tensors
// with d = 128 and B = 128 on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulate).
//
// One workgroup (4 waves, one per SIMD; two workgroups per compute unit) per (batch, head, query block m); it
// walks the compacted ascending list of selected key blocks of that row (or every n <= m for the dense baseline).
//
// Transposed products.  S^T = K Q^T and O^T = V^T P^T, so a lane always owns one QUERY (MFMA
// column = lane % 32): the softmax statistics of a query are per-lane scalars, and the fp32 S^T
// accumulators, rounded to bf16, already ARE the B operand of the second product -- P never goes
// through LDS.  The k-index order inside an MFMA is free as long as both operands agree, so V^T
// is laid out in LDS in exactly the key order in which the S^T accumulators hold the keys
// (0-3, 8-11 | 4-7, 12-15 of every 16).
//
// Work split.  Wave w owns the 32 queries 32 w .. +31 of the block and every key; a key block is walked as two
// tiles of 64 keys, a tile in two steps of 32.  Under this kernel the chip is power limited (the clock drops from
// 2.39 GHz to 1.7 GHz), so the time goes to whatever leaves the matrix pipe idle: the start of a row (order ->
// count -> list -> first tile, each waiting for the one before) and its end (diagonal block, output).  With 64 KB
// of tile buffers and at most 256 registers per lane TWO workgroups share a compute unit, and one's start and end
// run behind the other's tiles.
// Measured against one workgroup of 8 waves per compute unit with 128 KB of tile buffers (a wave then owned 32
// queries and one key half of a 128-key tile; the same MFMAs, LDS reads and copies per block), 32 / 8 heads, both on one
// machine: estimate + sparse 8K tokens 317 -> 256 us, 128K 35.6 -> 33.9 ms, 64K / 64 heads 24.9 -> 23.6 ms, dense 16K 2.15
// -> 2.01 ms, eight packed prompts 1.75 -> 1.49 ms.
// A launch that takes as long as its longest row is the other way round: it runs the row with both halves side by side
// (kWide; wide_rows_pay says when), the halves of a query merged in LDS at the end.
//
// Software pipeline.  On this chip the vector ALU instructions of a SIMD do not run in the shadow
// of its MFMAs for more than a few cycles per MFMA (measured: 32 MFMAs + the softmax of 32 scores
// take 1320 cycles against 975 for the MFMAs alone, with one or two waves per SIMD alike), but LDS
// reads, tile copies and scalar work do, so the steps are skewed: phase j issues the MFMAs of
// PV(step j-1) and QK(step j+1) interleaved with the softmax of step j, one element per
// MFMA slot.  The softmax itself is pipelined over the slots (scale, exp2, bf16 rounding and row sum of
// an element sit in four different slots), so that a wave never issues a vector instruction right behind
// the one that produces its operand.  The running maximum is lazy: P is taken relative to a reference that is only moved
// (with a rescale of O^T and the denominator) when a lane's terms add up to far more than the reference's, which
// keeps the common path branch-free (all terms of a row share the reference).
//
// Precision.  P is rounded to bf16 for the second product, and the denominator sums P as rounded: a row's weights add up
// to one, and the error of a large weight w weighs 1 - w.  (What rounding took from the diagonal block's terms and
// from those of a step that moved the reference is kept apart, for the log-sum-exp.)  A weight that the reference was
// moved to is 1 and exact, so a row is the more precise the less a weight may exceed the reference.  Error against 64 bits,
// 2-norm, of which the last rounding is 1.667e-3; moved beyond 2^8, 2^6, 2^5 (8 heads of 32):
//   4096 tokens 1.811e-3, 1.804, 1.796; 65536 tokens 1.841, 1.832, 1.825; dense, 16384 tokens 1.806, 1.801, 1.797
//   chunks: 1000 tokens at 20480 1.826, 1.810, 1.797; 2048 at 65536 1.853, 1.827, 1.812; 300 at 32768 1.890, 1.865, 1.844
//   64 tokens at 65536 1.805, 1.796, 1.792; ten chunks and steps 1.842, 1.825, 1.811 in the mean
// With two key halves to a row, each with a reference of its own moved beyond 2^8, and the diagonal block's terms summed
// unrounded: 1.816, 1.844, 1.816; 1.804, 1.825, 1.890; 1.805, 1.833.  2^8 stays below that for whole prompts and steps and 2^6
// for chunks, whose rows lie deep in the context.  A move is dear: 2^6 costs a chunk 1-2 %, 2^5 4-9 % and a prompt 1-3 %.
//
// Staging.  K and V tiles go global -> LDS directly (global_load_lds, 16 bytes per lane, no
// staging registers), row-major, double-buffered one key block ahead.  K fragments are plain
// 16-byte LDS reads; V^T fragments come out of the row-major V tile through the transposing LDS
// read (ds_read_b64_tr_b16: within 16 lanes, lane 4e+q supplies four consecutive d of key e and
// lane 4q+c receives element c of all four keys).  Each tile has its own XOR swizzle of the
// 16-byte chunks so that these reads are bank-conflict-free.
// The diagonal block (token-causal mask) is handled after the pipeline by a plain masked pass that skips
// the steps no query of the wave can see; its tile is fetched by the pipeline's last two copy slots.
//
// Lengths.  When the real length ends inside the last block (kRagged), that block is the only partial
// tile: it is read by the diagonal pass alone, through copies whose source rows stop at the last real
// position; query rows past the length work on a copy of the last real row and are not stored.
#include "rr_common.hpp"
#include "rr_attn_rows.hpp"
#include "rr_select.hpp"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace rr {

namespace {

constexpr int kWaves = 4;                            // 32 queries each
constexpr int kThreads = 64 * kWaves;
constexpr int kTileKeys = 64;
constexpr int kRowsPerWave = kTileKeys / kWaves;     // tile rows each wave copies
constexpr int kCopies = kRowsPerWave / 4;            // copy instructions per wave and tile (4 rows each)
constexpr int kTileBytes = kTileKeys * 256;          // one 64 x 128 bf16 tile
constexpr int kLdsBytes = 4 * kTileBytes;            // K and V, two stages each
constexpr int kOutRowBytes = 264;                    // 128 bf16 + 8 bytes of padding
constexpr int kXchgFloats = 67;                      // per lane, of a wide workgroup's second group: O^T, reference, sums

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((address_space(3))) unsigned char lds_byte_t;
typedef __attribute__((address_space(3))) int lds_int_t;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr_t;

__device__ __forceinline__ int k_swz(int key, int chunk) { return key * 256 + ((chunk ^ (key & 15)) << 4); }
__device__ __forceinline__ int v_swz(int key, int chunk) { return key * 256 + ((chunk ^ ((key & 7) << 1)) << 4); }

// workgroup id -> (batch, head, query block).  Workgroups are dealt to the 8 XCDs round-robin (id % 8 picks the XCD) and
// start in id order.
// Dense calls (by_group) as dense_order says: every XCD takes KV groups of its own (rr_attn_rows.hpp), so that the rows
// that run on it, which walk their blocks in the same order, find each other's tiles in its L2.  All groups cost the same
// there; XCDs that share a group take its rows in turn.  Against sets of groups over all XCDs (below; the order before
// where Nb is a multiple of 8, elsewhere level with what was), dense, us: 32 / 8 heads, 4096 tokens 157 / 147, 8192
// 533 / 512, 16384 2002 / 1946, 32768 7817 / 7506, 98304 67445 / 67180; four prompts of 16384 8014 / 7575, sixteen of 2048
// 686 / 623 (group after group; rank by rank of all an XCD's groups 7704, 635).
// Elsewhere, when Nb is a multiple of 8 the KV groups are taken `gi` at a time GPU-wide, so that the keys and values in use
// stay cache resident and L2 misses of the sparse walk stay off HBM (gi = 1 at 128K tokens, where one group's K and V are
// 64 MB); XCD x takes the rows with rank = x (mod 8), the query heads of a group back to back, rows heaviest (largest m)
// first.  Otherwise XCDs are given whole KV groups where the counts allow it.
// Interleaving.  Inside a set of gi groups the launch goes rank by rank, not group by group: every group's heaviest row,
// then every group's second, ...  Taken one after the other, each group would end with a tail of light rows that leaves
// compute units idle while the next group's heavy rows have not started; with few rows per compute unit (short contexts)
// those tails were a quarter of the launch.  The position of a group inside a rank rotates with the rank, so that an XCD is
// not always handed the same (perhaps heaviest) group.
// Ordered launches: the entry of the caller-supplied row order (rows of each KV group, heaviest first) that launch rank
// `bid` stands for, with the batch index and the first query head of its KV group.  Sets of gi groups, rank by rank inside
// a set, the group's position rotating with the rank.
__device__ __forceinline__ int order_entry_of(int bid, const Geom& g, int Nb, const int32_t* order, int gi, int hoist,
                                              int& b, int& h0) {
    const int N = g.G * Nb, NG = g.batch * g.Hkv;
    const bool first = bid < NG * hoist;                   // the `hoist` heaviest rows of every group, then the sets
    const int n = first ? NG : gi, rows = first ? hoist : N - hoist;
    const int at = first ? bid : bid - NG * hoist;
    const int set = at / (n * rows), r = at - set * (n * rows);
    const int q = r / n;
    const int rank = first ? q : hoist + q;
    const int grp = set * n + (r - q * n + rank) % n;
    b = grp / g.Hkv;
    h0 = (grp - b * g.Hkv) * g.G;
    return order[(long long)grp * N + rank];
}

__device__ __forceinline__ bool decode_block(int bid, const Geom& g, int Nb, const int32_t* order, int a_interleave, int hoist,
                                             int by_group, bool packed, int& b, int& h, int& m) {
    const int NG = g.batch * g.Hkv, G = g.G;
    int mr, grp, hl;
    if (order) {
        const int v = order_entry_of(bid, g, Nb, order, a_interleave, hoist, b, h);
        if ((unsigned)v >= (unsigned)(G * Nb)) return false;
        hl = v / Nb;
        m = v - hl * Nb;
        h += hl;
        return true;
    }
    if (by_group == kGroupByGroup && (NG & 7) == 0) {
        const RowPlace p = row_of_whole_groups(bid, G, Nb);
        grp = p.grp; hl = p.hl; mr = p.mr;
    } else if ((Nb & 7) == 0 && !by_group) {
        // one KV group after the other GPU-wide (its keys and values then fit the memory-side
        // cache); XCD x takes the rows with rank = x mod 8, the heads of a group back to back
        const int x = bid & 7, s = bid >> 3;
        hl = s % G;
        const int q = s / G, nb8 = Nb >> 3, gi = a_interleave;
        const int set = q / (gi * nb8), q2 = q - set * (gi * nb8);
        const int level = q2 / gi;                        // eight ranks of every group of the set, then the next eight
        grp = set * gi + (q2 - level * gi);
        // the residue an XCD takes rotates with the head: rows that are heavy in every head (the
        // protected last row keeps all blocks) are then spread over the XCDs instead of piling up on one
        mr = level * 8 + ((x + grp * G + hl) & 7);
    } else if ((NG & 7) == 0) {
        const RowPlace p = row_of_groups_by_rank(bid, NG, G);
        grp = p.grp; hl = p.hl; mr = p.mr;
    } else if (8 % NG == 0) {
        const RowPlace p = row_of_shared_group(bid, NG, G, Nb, packed);
        grp = p.grp; hl = p.hl; mr = p.mr;
    } else {
        mr = bid / (NG * G);
        const int r = bid - mr * NG * G;
        grp = r / G;
        hl = r - grp * G;
    }
    if (mr >= Nb) return false;
    m = Nb - 1 - mr;
    b = grp / g.Hkv;
    h = (grp - b * g.Hkv) * G + hl;
    return true;
}

__host__ unsigned grid_size(const Geom& g, int Nb, bool ordered) {
    const int NG = g.batch * g.Hkv;
    if (ordered) return (unsigned)NG * g.G * Nb;
    if ((Nb & 7) == 0) return (unsigned)NG * g.G * Nb;
    if ((NG & 7) != 0 && 8 % NG == 0) {
        const int k = 8 / NG;
        return 8u * g.G * ((Nb + k - 1) / k);
    }
    return (unsigned)NG * g.G * Nb;
}

#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// The MFMAs are one-instruction asm statements so that the register class of every operand is
// fixed by hand: O^T and the Q^T operand live in the accumulation registers (only the matrix
// pipe touches them), S^T lands in ordinary vector registers because the softmax reads it with
// vector ALU instructions.  (Left to itself the compiler puts every MFMA result in accumulation
// registers and copies S^T out and back around each instruction.)
// The compiler does not see inside these statements and adds no wait states for them.  The code
// keeps the distances itself: inside the pipeline a result is only reused as the accumulator of
// the next MFMA of its chain (which the matrix pipe interlocks) or, for S^T, read by vector
// instructions a whole phase and a barrier later; wherever else vector instructions touch a
// result, a settle statement comes first.
#define RR_MFMA_TEXT "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0"
__device__ __forceinline__ void mfma_pv(f32x16& acc, const bf16x8& vt, const bf16x8& pt) {
    asm volatile(RR_MFMA_TEXT : "+a"(acc) : "v"(vt), "v"(pt));
}
__device__ __forceinline__ void mfma_qk(f32x16& s, const bf16x8& k, const bf16x8& qt) {
    asm volatile(RR_MFMA_TEXT : "+v"(s) : "v"(k), "a"(qt));
}
__device__ __forceinline__ void mfma_qk_first(f32x16& s, const bf16x8& k, const bf16x8& qt) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(k), "a"(qt));
}
// Idle issue cycles longer than the tail of the last MFMA, then the values pass through empty
// asm statements: whatever reads them afterwards depends on those statements and therefore
// cannot be scheduled in front of the idle cycles.
__device__ __forceinline__ void mfma_settle_s(f32x16& s) {
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" : "+v"(s));
}
__device__ __forceinline__ void mfma_settle_acc(f32x16 (&acc)[4]) {
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15");
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) asm volatile("" : "+a"(acc[dt]));
}

// Per-wave state and operand addressing.
struct Wave {
    const lds_byte_t* lds;
    int lane, l32, gsel;
    float sl2;                         // log2(e) / sqrt(d)
    float lazy, lazy_sum;              // how far above the softmax reference a score may lie: in log2 units, and 2^ that
    bool tight;                        // a constant: no registers for two tiles of O^T outside their place, see move_reference
    bf16x8 qf[8];                      // Q^T operand: 16-wide d chunks
    f32x16 acc[4];                     // O^T: 32-row d tiles
    float mref;                        // softmax reference of the lane's query, log2 units
    float lsum;                        // this lane's part of the denominator: the sum of P as rounded
    float lfix;                        // what rounding took from it where that is known, for the log-sum-exp
    // Per-lane LDS byte addresses.  The XOR swizzle makes the chunk part of an address
    // base ^ (32 * kc) for K and base ^ (64 * dt) for V.
    unsigned ka0;                      // K: row lane%32, chunk gsel, swizzled
    unsigned va0;                      // V: keys 4 gsel + (lane%16)/4, d tile 0
    // ... and all of them, so that the hot loop forms no address: the chunk part is kaddr[kc] = ka0 ^ 32 kc,
    // vaddr[dt] = va0 ^ 64 dt; buffer, subtile and key-chunk selection ride in the instruction's immediate
    // offset (the loop is unrolled over the buffer parity for that).
    unsigned kaddr[8];
    unsigned vaddr[4];

    __device__ __forceinline__ void init_addresses() {
        const unsigned lds0 = (unsigned)(uintptr_t)lds;       // LDS addresses are 32 bits
        ka0 = lds0 + k_swz(l32, gsel);
        const int s16 = lane & 15, dhalf = (lane >> 4) & 1;
        const int key = 4 * gsel + (s16 >> 2);
        va0 = lds0 + 2 * kTileBytes + 8 * (s16 & 1) + v_swz(key, 2 * dhalf + ((s16 & 3) >> 1));
#pragma unroll
        for (int kc = 0; kc < 8; ++kc) kaddr[kc] = ka0 ^ (32u * kc);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) vaddr[dt] = va0 ^ (64u * dt);
    }
    __device__ __forceinline__ unsigned ka(int kc) const { return ka0 ^ (32u * kc); }
    __device__ __forceinline__ unsigned va(int dt) const { return va0 ^ (64u * dt); }
    __device__ __forceinline__ bf16x8 kfrag_at(unsigned at, int buf, int t) const {
        return *(const lds_bf16x8_t*)(uintptr_t)(at + (unsigned)(buf * kTileBytes + t * 32 * 256));
    }
    // fragment reads of the pipeline: address register + compile-time byte offset
    template <int OFF>
    __device__ __forceinline__ bf16x8 kfrag_imm(int kc) const {
        return *(const lds_bf16x8_t*)(uintptr_t)(kaddr[kc] + (unsigned)OFF);
    }
    template <int OFF>
    __device__ __forceinline__ bf16x8 vfrag_imm(int u) const { return vfrag_at(vaddr[u >> 1] + (unsigned)OFF, 0, 0, u); }
    __device__ __forceinline__ bf16x8 kfrag(int buf, int t, int kc) const { return kfrag_at(ka(kc), buf, t); }
    // V^T operand (32 d rows x 16 keys) of d tile u >> 1 and 16-key chunk u & 1 of subtile t: two
    // transposing reads, keys {4g..4g+3} and {8+4g..8+4g+3} of the chunk (accumulator order).
    __device__ __forceinline__ bf16x8 vfrag(int buf, int t, int u) const { return vfrag_at(va(u >> 1), buf, t, u); }
    __device__ __forceinline__ bf16x8 vfrag_at(unsigned at, int buf, int t, int u) const {
        const unsigned p = at + (unsigned)(buf * kTileBytes + t * 32 * 256 + (u & 1) * 16 * 256);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr_t)(uintptr_t)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr_t)(uintptr_t)(p + 8 * 256));
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, both);
    }
};

// S^T of one 32-key step, nothing overlapped (the diagonal block).
__device__ __forceinline__ void qk_step(const Wave& w, int buf, int t, f32x16& s) {
#pragma unroll
    for (int kc = 0; kc < 8; ++kc) {
        const bf16x8 kf = w.kfrag(buf, t, kc);
        if (kc == 0) mfma_qk_first(s, kf, w.qf[kc]);
        else mfma_qk(s, kf, w.qf[kc]);
    }
    mfma_settle_s(s);
}

// O^T += V^T P^T of one 32-key step, nothing overlapped.
__device__ __forceinline__ void pv_step(Wave& w, int buf, int t, const bf16x8 (&p)[2]) {
#pragma unroll
    for (int u = 0; u < 8; ++u) mfma_pv(w.acc[u >> 1], w.vfrag(buf, t, u), p[u & 1]);
    mfma_settle_acc(w.acc);
}

// P of a step's 16 scores against a reference: exp2, rounded; the sum of the rounded terms and of what rounding took.
__device__ __forceinline__ void exp_all(const Wave& w, const f32x16& s, float ref, bf16x8 (&p)[2], float& psum, float& fix) {
    const float nb = -ref;
    bf16x2 ones;
    ones[0] = (__bf16)1.0f;
    ones[1] = (__bf16)1.0f;
    float sum = 0.f;
    psum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
        const float e0 = __builtin_amdgcn_exp2f(fmaf(s[r], w.sl2, nb));
        const float e1 = __builtin_amdgcn_exp2f(fmaf(s[r + 1], w.sl2, nb));
        sum += e0;
        sum += e1;
        bf16x2 pr;
        pr[0] = (__bf16)e0;
        pr[1] = (__bf16)e1;
        p[r >> 3][r & 7] = pr[0];
        p[r >> 3][(r & 7) + 1] = pr[1];
        psum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, psum, false);
    }
    fix = sum - psum;
}
__device__ __forceinline__ float max_of(const f32x16& s) {
    float mx = -__builtin_huge_valf();
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
    return mx;
}

// Moves the softmax reference of the lane's query up to the new maximum, rescales O^T and the
// denominator, and recomputes P of the step at hand.  Rare; entered by the whole wave.  (Where registers are short, each
// tile of O^T is back in place before the next is taken; without that the ragged and persistent forms spill 12 to 25
// registers: 32K tokens 3357 against 3296 us.  The plain form has room, and is 0.7 % faster without: 64K, 64 heads.)
__device__ __forceinline__ void move_reference(Wave& w, const f32x16& s, bf16x8 (&p)[2], float& psum, float& fix, float mx) {
    mfma_settle_acc(w.acc);                             // O^T is about to be read by vector instructions
    float top = mx * w.sl2;
    top = fmaxf(top, __shfl_xor(top, 32));
    const float nref = fmaxf(w.mref, top);
    const float use = (nref == -__builtin_huge_valf()) ? 0.f : nref;
    const float alpha = __builtin_amdgcn_exp2f(w.mref - use);   // 0 while the reference is -inf
    w.mref = nref;
    w.lsum *= alpha;
    w.lfix *= alpha;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) w.acc[dt][r] *= alpha;
        if (w.tight) asm volatile("" : "+a"(w.acc[dt]));
    }
    exp_all(w, s, use, p, psum, fix);
    mfma_settle_acc(w.acc);                             // ... and was written by them
}

// softmax of one 32-key step, nothing overlapped (the diagonal block)
__device__ __forceinline__ void softmax_step(Wave& w, const f32x16& s, bf16x8 (&p)[2]) {
    float psum, fix;
    exp_all(w, s, w.mref, p, psum, fix);
    const float mx = max_of(s);
    if (__any(mx * w.sl2 > w.mref + w.lazy)) move_reference(w, s, p, psum, fix, mx);
    w.lsum += psum;
    w.lfix += fix;
}

// Global -> LDS copies of one 64 x 128 bf16 tile, kCopies instructions per wave (4 rows each), issued
// as asm statements: the compiler would otherwise make every later LDS read wait for them (it
// cannot tell that the reads go to the other buffer), which turns the prefetch into a blocking
// copy.  The kernel waits for them itself (wait_vm) before the barrier that hands a buffer over.
// Lane l lands in LDS slot (row l/16 of the group, physical chunk l%16) and therefore fetches
// logical chunk (l%16) ^ swizzle(row); the per-lane byte offsets of the wave's row groups are kept in
// registers, the tile origin is wave-uniform.
struct Stager {
    const unsigned short* Kp;
    const unsigned short* Vp;
    long long ksl;
    unsigned lds0;                     // LDS address of the buffers
    int wv;                            // wave index, uniform
    unsigned koff[kCopies];            // K: byte offset of this lane's 16 bytes in row group i
    unsigned voff[kCopies];            // V: same with the V swizzle

    __device__ __forceinline__ void init(int lane) {
        const int r4 = lane >> 4, c = lane & 15;
#pragma unroll
        for (int i = 0; i < kCopies; ++i) {
            const int row = 4 * i + r4;                    // row inside the wave's rows (16 | rows per wave: swizzle period)
            koff[i] = 2u * ((unsigned)(row * ksl) + 8u * (c ^ (row & 15)));
            voff[i] = 2u * ((unsigned)(row * ksl) + 8u * (c ^ ((row & 7) << 1)));
        }
    }
    // one of the copies of a tile: row group i of this wave's rows
    __device__ __forceinline__ void issue_one(const unsigned short* wave_src, unsigned wave_dst,
                                              const unsigned (&off)[kCopies], int i) const {
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                     :: "v"(off[i]), "s"(wave_src), "s"(wave_dst + 4 * i * 256) : "memory");
    }
    // this wave's rows of half `hf` (64 keys) of key block n
    __device__ __forceinline__ const unsigned short* k_src(int n, int hf) const {
        return Kp + ((long long)n * 128 + kTileKeys * hf + kRowsPerWave * wv) * ksl;
    }
    __device__ __forceinline__ const unsigned short* v_src(int n, int hf) const {
        return Vp + ((long long)n * 128 + kTileKeys * hf + kRowsPerWave * wv) * ksl;
    }
    __device__ __forceinline__ unsigned k_dst(int buf) const { return lds0 + buf * kTileBytes + kRowsPerWave * wv * 256; }
    __device__ __forceinline__ unsigned v_dst(int buf) const { return lds0 + (2 + buf) * kTileBytes + kRowsPerWave * wv * 256; }
    // Half `hf` of a block whose last rows lie past the real length (`rows` real rows, 1 <= rows < 128): those LDS
    // rows get a copy of the last real row (finite, and masked by token causality wherever a real query meets
    // them).  Offsets are formed on the spot from the block origin: this path runs once per launch row at most.
    __device__ __forceinline__ void issue_partial(const unsigned short* base, int n, int hf, unsigned dst, bool is_v,
                                                  int rows, int lane) const {
        const unsigned short* block = base + (long long)n * 128 * ksl;
        const int r4 = lane >> 4, c = lane & 15;
#pragma unroll
        for (int i = 0; i < kCopies; ++i) {
            const int row = 4 * i + r4;                      // LDS row inside the wave's rows: decides the swizzle
            const int src_row = min(kTileKeys * hf + kRowsPerWave * wv + row, rows - 1);
            const unsigned sw = is_v ? ((row & 7) << 1) : (row & 15);
            const unsigned off = 2u * ((unsigned)(src_row * ksl) + 8u * (c ^ sw));
            asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
                         :: "v"(off), "s"(block), "s"(dst + 4 * i * 256) : "memory");
        }
    }
    __device__ __forceinline__ void issue_k(int n, int hf, int buf) const {
#pragma unroll
        for (int i = 0; i < kCopies; ++i) issue_one(k_src(n, hf), k_dst(buf), koff, i);
    }
    __device__ __forceinline__ void issue_v(int n, int hf, int buf) const {
#pragma unroll
        for (int i = 0; i < kCopies; ++i) issue_one(v_src(n, hf), v_dst(buf), voff, i);
    }
};

__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// One pipeline phase: the MFMAs of PV(step j-1) [V^T fragments from LDS base vbase, operand pprev]
// and of QK(step j+1) [K fragments from kbase, result snext] interleaved with the exp2 / sum /
// max / bf16 rounding of step j [scores scur -> pcur], one element per MFMA slot, and (kFetch)
// with the wave's global -> LDS copies of the prefetched K and V tiles, one every other slot, so the
// copies never queue up in front of the arithmetic.  `valid` is false for the two fill phases at either end of a
// row, whose softmax is thrown away.
template <bool kFetch, int VOFF, int KOFF>
__device__ __forceinline__ void phase(Wave& w, const f32x16& scur, f32x16& snext,
                                      const bf16x8 (&pprev)[2], bf16x8 (&pcur)[2],
                                      bool valid, const Stager& st,
                                      const unsigned short* k_src, unsigned k_dst,
                                      const unsigned short* v_src, unsigned v_dst) {
    // The empty asm statements emit nothing.  Being ordered among themselves and with the MFMA
    // statements, they keep the compiler from sinking the softmax arithmetic out of the MFMA
    // shadow or hoisting all operand reads to the top.
    bf16x8 vf[2], kf[2];
    vf[0] = w.template vfrag_imm<VOFF>(0);
    kf[0] = w.template kfrag_imm<KOFF>(0);
    float psum = 0.f;
    const float nb = -w.mref;
    bf16x2 ones;
    ones[0] = (__bf16)1.0f;
    ones[1] = (__bf16)1.0f;
    // Softmax of step j, software pipelined over the MFMA slots so that no vector instruction waits for the
    // one in front of it: stage A (scale and shift of element k) runs at step k, B (its exp2) at step k + 1,
    // C (rounding the pair (2j, 2j+1) to bf16, which is what PV will use) at step 2j + 3, D (adding the pair to
    // the row sum) at step 2j + 4.
    constexpr int NE = 16;
    float tq[NE], ev[NE];
    auto step = [&](int sidx) {
        if (sidx >= 1 && sidx - 1 < NE) {                           // B
            ev[sidx - 1] = __builtin_amdgcn_exp2f(tq[sidx - 1]);
            asm volatile("" : "+v"(ev[sidx - 1]));
        }
        if (sidx < NE) {                                            // A
            tq[sidx] = fmaf(scur[sidx], w.sl2, nb);
            asm volatile("" : "+v"(tq[sidx]));
        }
        if (sidx >= 3 && (sidx & 1) && (sidx - 3) / 2 < NE / 2) {   // C
            const int er = sidx - 3;
            bf16x2 pr;
            pr[0] = (__bf16)ev[er];
            pr[1] = (__bf16)ev[er + 1];
            pcur[er >> 3][er & 7] = pr[0];
            pcur[er >> 3][(er & 7) + 1] = pr[1];
            asm volatile("" : "+v"(pcur[er >> 3]));
        }
        if (sidx >= 4 && !(sidx & 1) && (sidx - 4) / 2 < NE / 2) {  // D
            const int er = sidx - 4;
            bf16x2 pr;
            pr[0] = pcur[er >> 3][er & 7];
            pr[1] = pcur[er >> 3][(er & 7) + 1];
            psum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, psum, false);   // sums what PV will use
            asm volatile("" : "+v"(psum));
        }
    };
    // The scores of this step were completed by the last QK MFMA of the previous phase (an asm statement, so the
    // compiler adds no wait states for it); a vector instruction may read them 11 wait states after that MFMA
    // was issued.  The previous phase ends with a PV MFMA, which the matrix pipe accepts 8 wait states after
    // the QK one; the operand reads above and this statement add the rest whatever the compiler puts in
    // between.  The scores pass through the statement, so nothing that reads them can be scheduled in front.
    asm volatile("s_nop 2" : "+v"(const_cast<f32x16&>(scur)));
    // four steps run ahead of the first MFMA: they fill the softmax pipeline and cover the latency of the first
    // operand reads
    step(0);
    step(1);
    step(2);
    step(3);
    SCHED_FENCE();
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        // operand fragments of the next group are requested one group (2 MFMA slots) ahead
        if (u < 7) {
            vf[(u + 1) & 1] = w.template vfrag_imm<VOFF>(u + 1);
            kf[(u + 1) & 1] = w.template kfrag_imm<KOFF>(u + 1);
        }
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {
            // QK before PV: the phase then ends with a PV product, and the scores of the next step are complete
            // one MFMA earlier
            if (sl == 0) {
                if (u == 0) mfma_qk_first(snext, kf[0], w.qf[0]);
                else mfma_qk(snext, kf[u & 1], w.qf[u]);
                if (kFetch && (u & 1) == 0) st.issue_one(k_src, k_dst, st.koff, u >> 1);
                if (kFetch && (u & 1) == 1) st.issue_one(v_src, v_dst, st.voff, u >> 1);
            } else {
                mfma_pv(w.acc[u >> 1], vf[u & 1], pprev[u & 1]);
            }
            step(2 * u + sl + 4);
            SCHED_FENCE();
        }
    }
    // A score more than 2^8 (2^6) above the reference makes its term, hence the lane's sum of 16 terms,
    // exceed 2^8 (the first step of a row, whose reference is -inf, gives +inf): the sum is the
    // trigger, the maximum itself is only computed on the rare path.
    if (valid) {
        if (__any(!(psum <= w.lazy_sum))) {
            float fix;
            move_reference(w, scur, pcur, psum, fix, max_of(scur));
            w.lfix += fix;
        }
        w.lsum += psum;
    }
}

// Row queue of the persistent form: one counter per XCD, each on a cache line of its own, and one count of the
// workgroups that have left.  All zero between launches.
constexpr int kQueueStride = 16;                       // int32 words between counters
constexpr int kQueueDone = 8 * kQueueStride;

// The kernel's arguments as one struct, so that the persistent form can read them again from the kernel
// argument segment whenever it needs them instead of keeping ~50 scalar registers alive across its row loop
// (which pushed scalars into vector registers and those into scratch memory).
struct AttnKernelArgs {
    Geom g;
    AttnArgs a;
    float scale_log2;
    float lazy_log2, lazy_sum;
    unsigned starts;                   // persistent form, nibble q: of eight workgroups in a row, those that start with queue q
};
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) AttnKernelArgs* kernarg_ptr_t;
#else
typedef const AttnKernelArgs* kernarg_ptr_t;           // the host pass only parses the kernel
#endif
// the argument segment (the struct is the first and only argument, at offset 0); `fresh` hides from the compiler
// that it is the pointer it already knows, so that loads through it are made where they are written
template <bool kFresh>
__device__ __forceinline__ kernarg_ptr_t kernel_args() {
#if defined(__HIP_DEVICE_COMPILE__)
    kernarg_ptr_t p = (kernarg_ptr_t)__builtin_amdgcn_kernarg_segment_ptr();
    if (kFresh) asm volatile("" : "+s"(p));
    return p;
#else
    return nullptr;
#endif
}

template <bool kRagged, bool kPersist, bool kWide>
__global__ void __launch_bounds__(kWide ? 2 * kThreads : kThreads, 2)
k_attn_mfma_bf16(AttnKernelArgs kernel_arguments) {
    // kRagged: the real length ends inside the last block (g.Lr < g.L) or the queries start inside their first block
    // (g.qoff > 0): clamped Q rows, a clamped copy of the partial diagonal tile, predicated stores.  Compiled apart so that
    // the plain launch carries none of it (both forms run at the same rate).
    //
    // kPersist (sparse launches with a row order and a queue): two workgroups per compute unit that take row after row.  A
    // workgroup takes rows of one queue.  by_group, queue x mod NQ (x = workgroup mod 8, the XCD the dispatcher gave it; NQ
    // = min(groups, 8)) has the KV groups q, q + NQ, ..; else queue x has the launch ranks x + 8 t, so that every rank
    // keeps the XCD the order was made for.  The first rows go by workgroup index, the others are drawn from the queue's
    // counter, and the next row is looked up while the current one is merged and stored.  by_group, a workgroup whose queue
    // is empty goes on with the one that has the most rows left (groups differ in what they keep).
    //
    // kWide (launches whose time is that of a row, see launch_attn_mfma_bf16): two groups of four waves to a row, group hg
    // with the keys 64 hg .. +63 of every block and tile buffers of its own; one workgroup per compute unit (the persistent
    // form too).
    (void)kernel_arguments;
    extern __shared__ __align__(16) unsigned char lds_generic[];
    lds_byte_t* lds = (lds_byte_t*)lds_generic;
    const bool draws = threadIdx.x == 0;                    // the lane that talks to the row queue
    const float NEG_INF = -__builtin_huge_valf();

    // ---- the next row of a persistent workgroup ----
    // Fetched in five steps, each needing what the one before it loaded: (1) a ticket from the XCD's counter,
    // published to the other waves through LDS, (2) the entry of the row order that it stands for,
    // (3) the row, its count and its first list entry, (4) its last list entry, (5) done.  They are
    // placed in the tail of the current row: the ticket travels during the diagonal pass, the order entry during
    // the merge, count and first entry during the output stores; only the last entry is waited for.  The ticket
    // is deliberately NOT drawn earlier (say, at the
    // start of the row, which would hide all five steps): a workgroup that claims its next row a whole row
    // ahead starts it out of step with the rows queued around it, which were ordered to walk the same key
    // blocks at the same time on one XCD; measured, the early draw cost 2-3 % at 32K-128K tokens.
    struct NextRow {
        int rank;           // its place in the queue, or -1 when there is none
        int order_entry;    // as loaded
        bool live;          // the order entry names a row
        int b, h, mq;
        int count_raw, e0, elast;
    } nx;
    nx.rank = -1; nx.live = false; nx.order_entry = 0;
    nx.b = nx.h = nx.mq = 0; nx.count_raw = nx.e0 = nx.elast = 0;
    volatile lds_int_t* const ticket_slot = (volatile lds_int_t*)(lds + (kWide ? 2 : 1) * kLdsBytes);   // queue, place in it
    int queue_id = 0, ticket = 0;                           // lane 0 of wave 0
    auto groups_of = [&](const Geom& g, int q) {
        const int NG = g.batch * g.Hkv;
        return NG >= 8 ? (NG - q + 7) >> 3 : 1;
    };
    auto rows_of = [&](kernarg_ptr_t ka, const Geom& g, int q) {
        const int Nbq = g.Lq >> 7;
        return ka->a.by_group ? groups_of(g, q) * g.G * Nbq : (g.batch * g.Hq * Nbq - q + 7) >> 3;
    };
    auto first_of = [&](kernarg_ptr_t ka, int q) { return ((int)gridDim.x >> 3) * (int)((ka->starts >> (4 * q)) & 15u); };
    auto draw_issue = [&]() {
        if (draws) ticket = atomicAdd(kernel_args<true>()->a.queue + kQueueStride * queue_id, 1);
    };
    auto draw_publish = [&]() {                             // readable after the next workgroup barrier
        if (!draws) return;
        const kernarg_ptr_t ka = kernel_args<true>();
        const Geom g = ka->g;
        int at = first_of(ka, queue_id) + ticket;
        while (at >= rows_of(ka, g, queue_id)) {
            at = -1;
            if (!ka->a.by_group) break;
            // the queue with the most rows left (counters only grow: this ends)
            const int NQ = min(g.batch * g.Hkv, 8);
            int drawn[8], most = 0, from = -1;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                drawn[q] = q < NQ ? __hip_atomic_load(ka->a.queue + kQueueStride * q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int left = q < NQ ? rows_of(ka, g, q) - first_of(ka, q) - drawn[q] : 0;
                if (left > most) { most = left; from = q; }
            }
            if (from < 0) break;
            queue_id = from;
            at = first_of(ka, from) + atomicAdd(ka->a.queue + kQueueStride * from, 1);
        }
        ticket_slot[0] = queue_id;
        ticket_slot[1] = at;
    };
    auto step_order = [&](int q, int at) {                  // (2)
        const kernarg_ptr_t ka = kernel_args<true>();
        const Geom g = ka->g;
        const int Nbq = g.Lq >> 7;
        nx.live = false;
        nx.rank = -1;
        if (at < 0) return;
        nx.rank = at;
        int pb, ph;
        if (ka->a.by_group) {
            int grp = q, i = at;
            if (g.batch * g.Hkv > 8) {
                // the heaviest rows of all groups of the queue, then group by group
                const int n = groups_of(g, q), N = g.G * Nbq, hoist = ka->a.hoist;
                int gi;
                if (at < n * hoist) {
                    i = at / n;
                    gi = at - i * n;
                } else {
                    const int r = at - n * hoist;
                    gi = r / (N - hoist);
                    i = hoist + (r - gi * (N - hoist));
                }
                grp = q + 8 * gi;
            }
            pb = grp / g.Hkv;
            ph = (grp - pb * g.Hkv) * g.G;
            // The order is transposed inside runs of 8 G rows, for XCDs that take every eighth: here the rows as they were
            // sorted, the heads of a query block together (32 / 8 heads, 50000 tokens 7866 -> 7785 us; packed prompts of 311
            // blocks, 28 / 4, 1395 -> 1382).
            const int C = g.G, run = 8 * C;
            if (C > 1 && i < g.G * Nbq / run * run) {
                const int base = i / run * run, w = i - base;
                i = base + 8 * (w % C) + w / C;
            }
            nx.order_entry = ka->a.row_order[(long long)grp * (g.G * Nbq) + i];
        } else {
            nx.order_entry = order_entry_of(8 * at + q, g, Nbq, ka->a.row_order, ka->a.interleave, ka->a.hoist, pb, ph);
        }
        nx.b = __builtin_amdgcn_readfirstlane(pb);
        nx.h = __builtin_amdgcn_readfirstlane(ph);
    };
    auto step_rank = [&]() {
        const int q = __builtin_amdgcn_readfirstlane(ticket_slot[0]), at = __builtin_amdgcn_readfirstlane(ticket_slot[1]);
        step_order(q, at);
    };
    auto step_row = [&]() {                                 // (3)
        if (nx.rank < 0) return;
        const kernarg_ptr_t ka = kernel_args<true>();
        const int Nbq = ka->g.Lq >> 7;
        const int v = __builtin_amdgcn_readfirstlane(nx.order_entry);
        nx.live = (unsigned)v < (unsigned)(ka->g.G * Nbq);
        if (!nx.live) return;
        const int hl = v / Nbq;
        nx.mq = v - hl * Nbq;
        nx.h += hl;                                         // step_order left the group's first head here
        const long long rid = ((long long)nx.b * ka->g.Hq + nx.h) * Nbq + nx.mq;
        const int32_t* lp = ka->a.row_list + rid * ka->a.Nb;
        nx.count_raw = ka->a.row_count[rid];
        nx.e0 = lp[0];
    };
    auto step_last = [&]() {                                // (4)
        if (nx.rank < 0 || !nx.live) return;
        const kernarg_ptr_t ka = kernel_args<true>();
        const int Nbq = ka->g.Lq >> 7;
        // loaded values are the same in every lane: from here on they live in scalar registers
        nx.count_raw = __builtin_amdgcn_readfirstlane(nx.count_raw);
        nx.e0 = __builtin_amdgcn_readfirstlane(nx.e0);
        const int m = nx.mq + (ka->a.Nb - Nbq);
        int c = nx.count_raw;
        c = c < 0 ? 0 : (c > m + 1 ? m + 1 : c);
        const long long rid = ((long long)nx.b * ka->g.Hq + nx.h) * Nbq + nx.mq;
        int it = c > 0 ? c - 1 : 0;
        it = it < ka->a.Nb - 1 ? it : ka->a.Nb - 1;
        nx.elast = ka->a.row_list[rid * ka->a.Nb + it];
    };
    auto step_done = [&]() {                                // (5)
        if (nx.rank >= 0 && nx.live) nx.elast = __builtin_amdgcn_readfirstlane(nx.elast);
    };
    if (kPersist) {
        // the first row, by workgroup index: the same steps, each waiting for its loads
        const kernarg_ptr_t ka = kernel_args<false>();
        const int x = (int)blockIdx.x & 7, NQ = ka->a.by_group ? min(ka->g.batch * ka->g.Hkv, 8) : 8;
        queue_id = x % NQ;
        const int at = ((int)blockIdx.x >> 3) * (int)((ka->starts >> (4 * queue_id)) & 15u) + x / NQ;
        step_order(queue_id, at < rows_of(ka, ka->g, queue_id) ? at : -1);
        step_row(); step_last(); step_done();
    }

  constexpr bool kSplit = kRagged && !kPersist;              // the instantiations that also serve launches in parts
  for (;;) {
    // (The persistent form reads its arguments again for every row, and derives everything that depends on the
    // lane from a thread index the compiler takes for a new value each time: hoisted out of the row loop, the
    // lane's fragment, exchange and staging addresses stayed alive through all of it and spilled.)
    int tid = threadIdx.x;
    if (kPersist) asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int hg = kWide ? __builtin_amdgcn_readfirstlane(tid >> 8) : 0;                  // the wave's group
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6) - 4 * hg;                     // its place in that
    const kernarg_ptr_t kargs = kernel_args<kPersist>();
    const Geom g = kargs->g;
    const AttnArgs a = kargs->a;
    const float scale_log2 = kargs->scale_log2;
    // rows of the launch: the Lq / 128 query blocks of the call (chunked prefill: the last ones of the context)
    const int Nbq = g.Lq >> 7;
    int b, h, mq;
    bool have_row;
    int pf_count = 0, pf_e0 = 0, pf_elast = 0;
    if (kPersist) {
        if (nx.rank < 0) break;                             // the queue is empty: leave
        have_row = nx.live;
        b = nx.b; h = nx.h; mq = nx.mq;
        pf_count = nx.count_raw; pf_e0 = nx.e0; pf_elast = nx.elast;
    }
    // split launches: which share of the row's block list this workgroup walks
    int part = kSplit ? (int)blockIdx.x % a.nsplit : 0;
    bool split = kSplit && a.nsplit > 1;
    const bool planned = kSplit && a.split_len > 0;
    int plan_slot = -1;                                     // planned launches: where this part's result goes
    if (!kPersist) {
        // A planned launch has one workgroup per slot the plan could have used and one per row.  The slots in use
        // come first (the parts of the cut rows: the longest items of the launch), then the rows (a cut row's own
        // workgroup leaves at once), and the workgroups of unused slots last, where they leave while the others finish.
        const int grid_rows = planned ? (int)gridDim.x - a.split_budget : 0;
        const int used = planned ? __builtin_amdgcn_readfirstlane(*a.plan_total) : 0;
        if (planned && (int)blockIdx.x < used) {
            plan_slot = (int)blockIdx.x;
            const int rid = __builtin_amdgcn_readfirstlane(a.plan_items[plan_slot]);
            if ((unsigned)rid >= (unsigned)(g.batch * g.Hq * Nbq)) return;
            part = plan_slot - __builtin_amdgcn_readfirstlane(a.plan_row[rid]);
            if (part < 0) return;
            mq = rid % Nbq;
            const int bh = rid / Nbq;
            h = bh % g.Hq;
            b = bh / g.Hq;
            have_row = true;
        } else {
            const int rank = (int)blockIdx.x - used;
            if (planned && rank >= grid_rows) return;
            have_row = decode_block(kSplit && !planned ? rank / a.nsplit : rank, g, Nbq, a.row_order, a.interleave, a.hoist, a.by_group,
                                    a.seq_first != nullptr, b, h, mq);
            if (planned) part = 0;
        }
        if (!have_row) return;
    }
   if (have_row) {
    // the same for every lane: keep them (and all the addresses derived from them) in scalar registers
    b = __builtin_amdgcn_readfirstlane(b);
    h = __builtin_amdgcn_readfirstlane(h);
    mq = __builtin_amdgcn_readfirstlane(mq);
    const int m = mq + (a.Nb - Nbq);                    // query block inside the context: causal limit of the row

    Wave w;
    w.lds = lds + hg * kLdsBytes;
    w.lane = lane; w.l32 = lane & 31; w.gsel = lane >> 5;
    w.sl2 = scale_log2;
    w.lazy = kargs->lazy_log2;
    w.lazy_sum = kargs->lazy_sum;
    w.tight = kRagged || kPersist;
    w.init_addresses();
    const int l32 = w.l32, gsel = w.gsel;
    const int kv = h / g.G;
    const long long row_id = ((long long)b * g.Hq + h) * Nbq + mq;
    const unsigned short* Qp = reinterpret_cast<const unsigned short*>(a.Q) + b * g.qsb + h * g.qsh;
    Stager st;
    st.Kp = reinterpret_cast<const unsigned short*>(a.K) + b * g.ksb + kv * g.ksh;
    st.Vp = reinterpret_cast<const unsigned short*>(a.V) + b * g.ksb + kv * g.ksh;
    st.ksl = g.ksl;
    st.lds0 = (unsigned)(uintptr_t)w.lds;
    st.wv = wv;
    st.init(lane);

    // a caller-made list is not trusted with addresses: the count is held to [0, m+1] and entries to [0, m]
    // (a list that breaks the contract gives a wrong row, never an access outside K and V)
    // the dense walk starts at block 0, or (packed sequences) at the first block of the row's sequence
    int first_in = (!a.row_list && a.seq_first) ? a.seq_first[m] : 0;
    first_in = first_in < 0 ? 0 : (first_in > m ? m : first_in);
    const int first = __builtin_amdgcn_readfirstlane(first_in);
    int count_in = kPersist ? pf_count : (a.row_list ? a.row_count[row_id] : (m + 1 - first));
    count_in = count_in < 0 ? 0 : (count_in > m + 1 ? m + 1 : count_in);
    int count = __builtin_amdgcn_readfirstlane(count_in);
    // a split launch: entries [list_lo, list_lo + count) of the row's list are this workgroup's; the diagonal
    // block (always the last entry) belongs to the part that holds the end of the list
    int list_lo = 0;
    bool last_part = true;
    if (planned) {
        // the plan decides: a row without slots is an ordinary row that stores its own result
        const int base = __builtin_amdgcn_readfirstlane(a.plan_row[row_id]);
        split = base >= 0;
        if (split != (plan_slot >= 0)) return;              // a cut row is computed by its slots' workgroups only
        if (split && plan_slot != base + part) return;
    }
    if (split) {
        int hi;
        if (planned) {
            const int len = __builtin_amdgcn_readfirstlane(a.plan_total[2]), parts = (count + len - 1) / len;
            if (part < (parts & ~7)) {
                // The heads of a KV group whose last query block keeps every block, two thirds of such a launch, walk the same
                // ranges of keys: part p goes to the XCD p mod 8 in every row, where the tiles of the others may still be in L2.
                // 2048 tokens at 128K: estimate and attention 621 -> 590 us, L2 hit rate 17 -> 42 % (44 % with the equal parts).
                const int taken = (part & ~7) + ((int)blockIdx.x & 7);
                plan_slot += taken - part;
                part = taken;
            }
            list_lo = count * part / parts;                 // equal parts: dense, 2048 tokens at 128K 4.36 -> 3.82 ms
            hi = count * (part + 1) / parts;
        } else {
            const int len = (count + a.nsplit - 1) / a.nsplit;
            list_lo = min(count, part * len);
            hi = min(count, list_lo + len);
        }
        last_part = hi == count;
        count = hi - list_lo;
    }
    const int32_t* list = a.row_list ? a.row_list + row_id * a.Nb + list_lo : nullptr;
    // entry `it` of the row's block list (clamped: entries are read ahead of their use); the value is
    // the same in every lane, block_at() moves it to a scalar register
    const int tile_rows = g.Lr - m * 128;               // real rows of block m; < 128 only for a partial last block
    const bool partial = kRagged && tile_rows < 128;
    auto clamp_block = [&](int n) { return n < 0 ? 0 : (n > m ? m : n); };
    auto block_raw = [&](int it) {
        it = it < a.Nb - 1 - list_lo ? it : a.Nb - 1 - list_lo;
        return clamp_block(list ? list[it] : first + list_lo + it);
    };
    // the entries a row needs before its first tile: the first and the last (the persistent form has them already)
    const int e0_raw = kPersist ? clamp_block(pf_e0) : block_raw(0);
    const int e1_raw = kWide ? block_raw(1) : 0;
    const int elast_raw = kPersist ? clamp_block(pf_elast) : block_raw(count > 0 ? count - 1 : 0);
    // the diagonal block, if listed, is the last entry; it is taken after the pipelined blocks
    const bool has_diag = last_part && count > 0 && __builtin_amdgcn_readfirstlane(elast_raw) == m;
    const int cnt = count - (has_diag ? 1 : 0);

    // ---- Q^T operand: this lane's query, d = 16*kc + 8*gsel .. +7 ----
    {
        // (query rows that do not exist -- past the real length, or in front of a step that starts inside its
        // first block -- work on a copy of the nearest real row)
        int row_in = mq * 128 + 32 * wv + l32;
        if (kRagged) row_in = max(min(row_in - g.qoff, g.Lr - g.q0 - 1), 0);
        const long long row = row_in;
#pragma unroll
        for (int kc = 0; kc < 8; ++kc)
            w.qf[kc] = *reinterpret_cast<const bf16x8*>(Qp + row * g.qsl + 16 * kc + 8 * gsel);
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) w.acc[dt][r] = 0.f;
    w.mref = NEG_INF;
    w.lsum = 0.f;
    w.lfix = 0.f;

    f32x16 sa, sb;
    bf16x8 pa[2], pb[2];
    const bool ahead = cnt > 0 && has_diag && !partial;      // the pipeline brings the diagonal block in

    if (cnt > 0) {
        // Tiles tau = 2 i + hf (half hf of the row's i-th pipelined block), steps j = 2 tau + t; K(tau) and V(tau)
        // sit in buffers tau & 1 = hf.  Tile iteration tau runs phases 2 tau + 1 and 2 tau + 2, which use K(tau+1)
        // and V(tau), and fetches K(tau+2) and V(tau+1) behind its barrier.  The same code also fills and drains
        // the pipeline: iteration -1 computes S(0) and the softmax of step 0 (its PV products use a
        // zero P against the K(0) tile, which is there and finite), iteration 2 cnt - 1 finishes the
        // last PV products (its QK products are those of the diagonal block's first half, or of whatever the idle
        // K buffer holds, and are then never used).
        // A wide workgroup's group walks one tile to a block, its own half: tile tau = i, in buffers tau & 1.
        int n_next = __builtin_amdgcn_readfirstlane(e0_raw);     // block i + 1 of trip i
        // A partial block m is only ever read by the diagonal pass, whose copies stay inside the real length:
        // an entry of a malformed list that names it in the middle of the row is moved to block m - 1.
        // Applied to the scalar copy of an entry, where it is consumed: touching the loaded value any earlier
        // would move the wait for the list load, and with it a stall, into the middle of the iteration.
        auto whole_tile = [&](int n) { return (partial && n == m && m > 0) ? m - 1 : n; };
        n_next = whole_tile(n_next);
        st.issue_k(n_next, hg, 0);
        wait_vm();
        // The Q^T operand must be complete in its registers here.  Its loads may target the accumulation
        // registers directly, and their first reader would then be an MFMA inside the tile loop: the compiler
        // places its waits for the eight loads there (vmcnt(7) .. vmcnt(0) in front of successive MFMAs), and
        // on every later trip those same waits stall on the tile copies in flight instead -- 6 % of the launch.
#pragma unroll
        for (int kc = 0; kc < 8; ++kc) asm volatile("" : "+a"(w.qf[kc]));
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) { pa[c][e] = (__bf16)0.f; pb[c][e] = (__bf16)0.f; }
        // The copies being unconditional, the pipeline fetches one block (less its second V half) past its last.
        // With a whole diagonal block selected that is this block (list entry cnt); otherwise the last one again.
        const int last_entry = ahead ? cnt : cnt - 1;
        auto entry_raw = [&](int it) { return block_raw(it < last_entry ? it : last_entry); };
        int n_cur = n_next;
        // One tile iteration; HF is a compile-time constant so that every LDS offset is an immediate.  `fill`
        // marks iteration -1, which only starts the pipeline: it computes S(0),
        // S(1) and the softmax of step 0; its PV products multiply whatever the idle V buffer holds and are
        // thrown away by clearing O^T afterwards.  (The fill must stay an ordinary trip of the one loop: peeled
        // off, the compiler knows O^T to be zero there, builds the accumulator tuples of the asm MFMAs from
        // copies and moves the results right behind each MFMA without the wait states an MFMA result needs.)
        auto tile = [&](auto half, bool fill, bool more, int nk, int nv) {
            constexpr int HF = decltype(half)::value;                  // tau & 1
            constexpr int KO = (HF ^ 1) * kTileBytes;
            constexpr int VO = HF * kTileBytes;
            // phase 2 tau + 1: softmax | PV(2 tau) QK(2 tau + 2) | fetch K(tau+2) of block nk and V(tau+1) of block nv
            phase<true, VO, KO>(w, sb, sa, pa, pb, !fill, st, st.k_src(nk, kWide ? hg : HF), st.k_dst(HF),
                                st.v_src(nv, kWide ? hg : HF ^ 1), st.v_dst(HF ^ 1));
            // phase 2 tau + 2: softmax | PV(2 tau + 1) QK(2 tau + 3)
            phase<false, VO + 32 * 256, KO + 32 * 256>(w, sa, sb, pb, pa, more, st, nullptr, 0, nullptr, 0);
        };
        auto clear_acc = [&]() {
            mfma_settle_acc(w.acc);
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) w.acc[dt][r] = 0.f;
            mfma_settle_acc(w.acc);
        };
        using std::integral_constant;
        if constexpr (kWide) {
            int n2 = whole_tile(__builtin_amdgcn_readfirstlane(last_entry >= 1 ? e1_raw : e0_raw));   // block i + 2 of trip i
            auto iteration = [&](int i, auto parity, bool fill) {
                __syncthreads();
                const int n3_raw = entry_raw(i + 3);                  // requested in front of the copies, as below
                tile(parity, fill, i + 1 < cnt, n2, n_next);
                if (fill) clear_acc();
                wait_vm();
                n_next = n2;
                n2 = whole_tile(__builtin_amdgcn_readfirstlane(n3_raw));
            };
            for (int i = -1; i < cnt; i += 2) {
                iteration(i, integral_constant<int, 1>{}, i < 0);
                if (i + 1 < cnt) iteration(i + 1, integral_constant<int, 0>{}, false);
            }
        } else {
            for (int i = -1; i < cnt; ++i) {
                if (i >= 0) {
                    __syncthreads();
                    tile(integral_constant<int, 0>{}, false, true, n_next, n_cur);
                    wait_vm();
                }
                __syncthreads();
                // list entry i + 2, wanted at the end of this trip: requested in front of the tile copies, so that it
                // is back long before the wait for them (loads complete in order)
                const int n2_raw = entry_raw(i + 2);
                tile(integral_constant<int, 1>{}, i < 0, i + 1 < cnt, n_next, n_next);
                if (i < 0) clear_acc();
                wait_vm();
                n_cur = n_next;
                n_next = whole_tile(__builtin_amdgcn_readfirstlane(n2_raw));
            }
        }
        mfma_settle_acc(w.acc);
        mfma_settle_s(sa);
        mfma_settle_s(sb);
    }

    if (kPersist) draw_issue();                             // (1): the ticket is back when the diagonal pass is done
    if (has_diag) {
        // ---- diagonal block: token-causal mask, no overlap inside the wave.  Wave w sees the 32-key steps 0 .. w,
        // the last of them through the mask.  Half hf sits in buffers hf; after the pipeline S of the first half
        // is in sa and sb already, and only the second half of V is still to come. ----
        __syncthreads();                                    // the pipeline is done; its last copies have landed
        // buffers of half hf
        auto buffer_of = [&](int hf) { return kWide ? (ahead ? cnt & 1 : 0) : hf; };
        if (!ahead) {
#pragma unroll
            for (int k = 0; k < (kWide ? 1 : 2); ++k) {
                const int hf = kWide ? hg : k;
                if (partial) {
                    st.issue_partial(st.Kp, m, hf, st.k_dst(buffer_of(hf)), false, tile_rows, lane);
                    st.issue_partial(st.Vp, m, hf, st.v_dst(buffer_of(hf)), true, tile_rows, lane);
                } else {
                    st.issue_k(m, hf, buffer_of(hf));
                    st.issue_v(m, hf, buffer_of(hf));
                }
            }
            wait_vm();
            __syncthreads();
        } else if (!kWide) {
            st.issue_v(m, 1, 1);
        }
        auto scores = [&](int j, f32x16& s) { qk_step(w, buffer_of(j >> 1), j & 1, s); };
        auto diag_step = [&](int j, f32x16& s) {            // 32-key step j of the block
            if (j == wv) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r >> 2) + 4 * gsel + (r & 3) > l32) s[r] = NEG_INF;
            }
            softmax_step(w, s, pa);
            pv_step(w, buffer_of(j >> 1), j & 1, pa);
        };
        // the steps of the first half, or of the group's own one
        if (!ahead && 2 * hg <= wv) {
            scores(2 * hg, sa);
            if (2 * hg + 1 <= wv) scores(2 * hg + 1, sb);
        }
        if (2 * hg <= wv) diag_step(2 * hg, sa);
        if (2 * hg + 1 <= wv) diag_step(2 * hg + 1, sb);
        if (!kWide) {
            if (ahead) {
                wait_vm();
                __syncthreads();
            }
            if (wv >= 2) {
                scores(2, sa);
                diag_step(2, sa);
            }
            if (wv >= 3) {
                scores(3, sb);
                diag_step(3, sb);
            }
        }
    }
    if (kPersist) draw_publish();
    __syncthreads();
    if (kPersist) step_rank();                              // (2): the order entry arrives during the normalisation

    // ---- a wide workgroup: the second group hands its half over; normalise, write ----
    float l = w.lsum + __shfl_xor(w.lsum, 32);
    float whole = l + (w.lfix + __shfl_xor(w.lfix, 32));
    float* const xch = reinterpret_cast<float*>(lds_generic) + wv * (kXchgFloats * 64) + lane;     // the tile buffers are free
    float f0 = 1.f, f1 = 0.f;                               // weights of the two halves
    if constexpr (kWide) {
        if (hg == 1) {
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) xch[(dt * 16 + r) * 64] = w.acc[dt][r];
            xch[64 * 64] = w.mref;
            xch[65 * 64] = l;
            xch[66 * 64] = whole;
        }
        __syncthreads();
        if (hg == 0) {
            const float m0 = w.mref, m1 = xch[64 * 64];
            const float mm = fmaxf(m0, m1);
            f0 = m0 == NEG_INF ? 0.f : __builtin_amdgcn_exp2f(m0 - mm);
            f1 = m1 == NEG_INF ? 0.f : __builtin_amdgcn_exp2f(m1 - mm);
            l = l * f0 + xch[65 * 64] * f1;
            whole = whole * f0 + xch[66 * 64] * f1;
            w.mref = mm;
        }
    }
    if (hg == 0) {
        const float inv = l > 0.f ? 1.0f / l : 0.f;
        const float w0 = kWide ? f0 * inv : inv, w1 = f1 * inv;
        unsigned char* ost = lds_generic + (kWide ? kWaves * kXchgFloats * 256 : 0) + wv * (32 * kOutRowBytes);
        // row of Q / O of this wave's first query (negative in front of a step that starts inside its first
        // block), and the rows of the wave that exist: rows_lo <= x < rows_q (may be empty in the ragged form)
        const long long wrow0 = (long long)mq * 128 + 32 * wv - (kRagged ? g.qoff : 0);
        const int rows_q = kRagged ? (int)min((long long)32, (long long)(g.Lr - g.q0) - wrow0) : 32;
        const int rows_lo = kRagged ? (int)max(0ll, -wrow0) : 0;
        // a split launch writes its part's result (normalised over the part's own blocks) and lse to the
        // workspace, rows contiguous; the merge kernel weighs the parts by their lse
        const long long rows_call = g.Lr - g.q0;
        float* lse_base = split ? a.part_lse + (long long)part * g.batch * g.Hq * rows_call : a.lse;
        float* lse = lse_base ? lse_base + ((long long)b * g.Hq + h) * rows_call + wrow0 : nullptr;
        if (planned && split) lse = a.part_lse + (long long)plan_slot * 128 + 32 * wv;   // a slot holds a whole tile
        if (lse && gsel == 0 && l32 < rows_q && l32 >= rows_lo)
            lse[l32] = l > 0.f ? w.mref * 0.6931471805599453f + logf(whole) : NEG_INF;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = w.acc[dt][4 * rg + e] * w0;
                    if (kWide) v[e] = fmaf(xch[(dt * 16 + 4 * rg + e) * 64], w1, v[e]);
                }
                if (split) {
                    // a part's result stays fp32 (the merge rounds once, at the end): straight from the
                    // registers, 16 bytes per lane
                    if (l32 < rows_q && l32 >= rows_lo) {
                        float* dst = planned
                            ? a.part_O + ((long long)plan_slot * 128 + 32 * wv + l32) * g.d + 32 * dt + 8 * rg + 4 * gsel
                            : a.part_O + (((long long)part * g.batch * g.Hq + (long long)b * g.Hq + h) * rows_call +
                                          wrow0 + l32) * g.d + 32 * dt + 8 * rg + 4 * gsel;
                        *reinterpret_cast<f32x4*>(dst) = f32x4{v[0], v[1], v[2], v[3]};
                    }
                } else {
                    u32x2 o = {f32_to_bf16_bits(v[0]) | (f32_to_bf16_bits(v[1]) << 16),
                               f32_to_bf16_bits(v[2]) | (f32_to_bf16_bits(v[3]) << 16)};
                    *reinterpret_cast<u32x2*>(ost + l32 * kOutRowBytes + 2 * (32 * dt + 8 * rg + 4 * gsel)) = o;
                }
            }
        if (kPersist) step_row();                           // (3): the order entry came in during the normalisation
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        unsigned short* Op = reinterpret_cast<unsigned short*>(a.O) + b * g.qsb + h * g.qsh + wrow0 * g.qsl;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int idx = lane + 64 * k, row = idx >> 4, ch = idx & 15;
            const u32x2 lo = *reinterpret_cast<const u32x2*>(ost + row * kOutRowBytes + 16 * ch);
            const u32x2 hi = *reinterpret_cast<const u32x2*>(ost + row * kOutRowBytes + 16 * ch + 8);
            u32x4 o = {lo[0], lo[1], hi[0], hi[1]};
            if (!split && row < rows_q && row >= rows_lo) *reinterpret_cast<u32x4*>(Op + (long long)row * g.qsl + 8 * ch) = o;
        }
        if (kPersist) step_last();                          // (4): count and first entry came in during the stores
    } else if (kPersist) {
        step_row();                                         // the waves that only handed their half over: (3), (4)
        step_last();
    }
   }  // have_row
    if (!kPersist) break;
    // what is left of the look-ahead (all of it after a rank without a row).  The barrier keeps the next row's
    // tile copies behind this row's last reads of the staging area.
    if (!have_row) { draw_issue(); draw_publish(); }
    __syncthreads();
    if (!have_row) {
        step_rank();
        // The next draw may be published before another barrier is met (the next rank may have no row either, or a row
        // without a block): not until every wave has read this ticket.
        __syncthreads();
        step_row();
        step_last();
    }
    step_done();                                            // (5)
  }
    if (kPersist && draws) {
        // every workgroup has drawn its last (empty) ticket before it counts itself out: the last one out
        // leaves the queue as it found it
        int32_t* const queue = kernel_args<true>()->a.queue;
        const int gone = atomicAdd(queue + kQueueDone, 1);
        if (gone == (int)gridDim.x - 1) {
#pragma unroll
            for (int x = 0; x < 8; ++x) queue[kQueueStride * x] = 0;
            queue[kQueueDone] = 0;
        }
    }
}

}  // namespace

constexpr int kPersistMaxBlocks = 256;                 // contexts up to 32K tokens, see launch_attn_mfma_bf16

// The order of launches that do not take their rows by KV group (by_group in launch_attn_mfma_bf16): the rules from here to
// hoisted_rows are for launches without a queue, with too few rows for it, or whose groups' keys and values do not fit the
// memory-side cache.  With a queue nearly all shapes of the three tables are taken by group now; their figures are those of
// rows in rank order, drawn from a queue per XCD up to 256 blocks and one workgroup to a row beyond.
//
// Whether the heaviest rows of all KV groups, one run of each group's row order (8 G rows, which one XCD each was chosen
// for), may go in front of the sets: up to 64 heads in all, whose runs are no more than the 512 workgroups that run at
// once, or up to 128 heads of long prompts, whose runs are at most a sixteenth of the rows, unless the rows of a group are
// many.  More of them are a visible share of the launch, mixed rows of many groups find less in L2, and the last set of a
// launch of many sets is a small part of it.  Estimate and attention with the runs in front / without, us, gain of the
// inputs 3, tau 0.9:
//   not taken: 64 / 8 heads, four prompts of 5000 tokens 902 / 857, of 12000 3674 / 3503, two of 9200 1130 / 1112, of 14000
//     2347 / 2290, of 30000 9290 / 9213 (on another box 9657 / 9741), of 40000 16271 / 15879 (17025 / 17221); 32 / 8, four
//     of 3000 229 / 221, of 9000 1153 / 1115, of 16000 3016 / 2976, eight of 6000 1251 / 1205, of 20000 9342 / 9221;
//     28 / 4, four of 10000 1196 / 1167, three of 36000 8677 / 8430; 8 / 2, sixteen of 8000 1016 / 979
//   taken: 32 / 8, four of 18500 3743 / 3964, 24000 6298 / 6509, 33000 11314 / 11824, 45000 21541 / 21344 (22369 / 22346);
//     64 / 8, two of 20000 4379 / 4393, 26000 7102 / 7167; 28 / 4, four of 20000 3899 / 3794, 25000 5704 / 5862; 16 / 4,
//     eight of 24000 6298 / 6480; 8 / 2, sixteen of 20000 4631 / 4772
bool first_runs_pay(const Geom& g) {
    const long long heads = (long long)g.batch * g.Hq;
    const int Nbq = g.Lq / 128;
    return heads <= 64 || (heads <= 128 && Nbq >= 128 && g.G * Nbq <= 1750);
}

// KV groups launched interleaved (decode_block, order_entry_of): the largest divisor of the number of groups that keeps K
// and V of the set within 32 MB, the L2 capacity of the chip (8 x 4 MB), or within 38 MB for the row order of whole prompts
// where the first runs pay and sets are at most 3000 rows long.  More groups to a set find less of each other's tiles in
// L2, fewer put more of a launch's heavy rows late, which counts where there are few sets and they are over soon.
// Measured, estimate and attention or dense call, us, 38 MB / 32 MB, gain of the inputs 3 and tau 0.9 unless said:
//   sets of up to 3000 rows: 32 / 8 heads, 18000 tokens 752 / 772, 37000 2772 / 2848; 16 / 4, 37000 1552 / 1736, tau 0.95
//     2168 / 2318; 8 / 2, 36000 810 / 873, 38900 883 / 931 (weaker structure, tau 0.95, 38500 1709 / 1670; three packed
//     prompts of 300 blocks 715 / 706)
//   longer ones (32 MB): 64 / 8, 9000 538 / 520, 18000 1747 / 1725, 35000 5092 / 4881, 38500 7564 / 7389; 28 / 4, 17000
//     708 / 699, 18500 647 / 653, 35000 2631 / 2587, 38000 3116 / 3056, packed prompts of 290 blocks 1286 / 1257
//   many short prompts (32 MB): 32 / 8, three of 12000 1402 / 1368, four of 9000 1118 / 1109
//   no row order or not a whole prompt (32 MB): dense, 32 / 8, 38900 11363 / 11119, 8900 to 36000 level; planned chunks,
//     1000 of 35000, 64 / 8 heads, 415 / 402 and 424 / 412, 1500 of 18500, 32 / 8, 209 / 203 and 200 / 203; sparse without
//     a row order level
int interleave_groups(const Geom& g, bool ordered) {
    const long long per_group = 2ll * g.L * g.d * 2;               // K and V of one KV head, bf16
    const int NG = g.batch * g.Hkv, rows = g.G * (g.Lq / 128);
    int gi = 1;
    for (int c = 1; c <= NG && c <= 64; ++c) {
        const bool more = ordered && g.q0 == 0 && first_runs_pay(g) && c * rows <= 3000;
        if (NG % c == 0 && c * per_group <= (more ? 38ll : 32ll) << 20) gi = c;
    }
    return gi;
}
// What starts late counts: the longest row (the protected one keeps every block) of the last set took as long as that whole
// set, so sparse launches first take the heaviest rows of ALL groups, one run of the row order, and then the sets.
// Not taken where
// - first_runs_pay says no
// - sets have 4096 rows and more (eight to each of the 512 workgroups that run at once), where it is even: 131072 tokens,
//   32 / 8 heads, with it 0.2 and 0.4 % slower in two runs, at weaker structure 0.4 and 1.1 %, at tau 0.95 0.7 and 0.6 %; 65536,
//   64 / 8, S = 8, 1.2 and 1.1 % faster, 65500, tau 0.95, 0.6 and 0.9 %
// - contexts of more than 256 blocks have fewer than eight groups: the last set is a large part of the launch there, and the
//   mixed rows cost what they save.
// Measured, attention alone, tau 0.9, us; sets of 32 MB without the first run / sets of 1, 2, 4 groups with it:
//   32 / 8 heads: 9000 tokens 265 / 208, 206, 206; 16384 628 / 580, 555, 541; 24000 1330 / 1217, 1171, 1158; 28000 1730 / 1580,
//     1532, 1545; 36000 3020 / 2699, 2643, 2736; 50000 4950 / 4637, 4617, 4731; 65536 8350 / 7906, 7704, 8065 (weaker structure
//     14349 / 14201, 14321, 15066); 98304 18126 / 18141, 18479, 19748
//   64 / 8: 12000 685 / 706, 694, 689; 20000 1704 / 1692, 1633, 1664
//   28 / 4: 20000 806 / 773, 731, 739; 8 / 2: 20000 272 / 260, 271; not taken: 28 / 4 40000 2715 / 2672; 8 / 2 50000 1204 / 1226;
//     28 / 4, eight packed prompts (311 blocks) 1371 / 1385
int hoisted_rows(const Geom& g, int interleave) {
    const int NG = g.batch * g.Hkv, rows = g.G * (g.Lq / 128);
    if (!first_runs_pay(g) || interleave == NG || interleave * rows >= 4096 || 8 * g.G >= rows ||
        (g.L / 128 > kPersistMaxBlocks && NG < 8))
        return 0;
    return 8 * g.G;
}

// compute units of the present device, a multiple of 8 so that workgroup i of a persistent launch sits on XCD i mod 8
int compute_units() {
    static std::atomic<int> cached[64];                    // zero-initialised; per device, written once
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        n = n / 8 * 8;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// ---- split launches: merge of the parts ----
// Every part holds softmax attention over its own key blocks, O_p and lse_p = log of its sum of exponentials; over
// all blocks O = sum_p exp(lse_p - lse) O_p with lse = log sum_p exp(lse_p) (Sec. 2.1: the softmax is one sum
// over the selected keys).  One wavefront per query row, a lane two channels of d = 128.
__global__ void __launch_bounds__(256)
k_attn_combine(Geom g, AttnArgs a) {
    const long long rows_call = g.Lr - g.q0;
    const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const long long nrows = (long long)g.batch * g.Hq * rows_call;
    if (row >= nrows) return;
    const int lane = threadIdx.x & 63;
    const long long bh = row / rows_call, r = row - bh * rows_call;
    const int b = (int)(bh / g.Hq), h = (int)(bh - (long long)b * g.Hq);
    const float NEG_INF = -__builtin_huge_valf();
    float mx = NEG_INF;
    for (int p = 0; p < a.nsplit; ++p) mx = fmaxf(mx, a.part_lse[(long long)p * nrows + row]);
    float den = 0.f, o0 = 0.f, o1 = 0.f;
    if (mx != NEG_INF) {
        // up to eight parts requested at once (one after the other, 64 tokens of 65536 133 -> 127 us in all), no more than there are
        int p0 = 0;
        auto take = [&](auto n) {
            constexpr int N = decltype(n)::value;
            float2 v[N];
            float l[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const long long at = (long long)min(p0 + u, a.nsplit - 1) * nrows + row;
                l[u] = a.part_lse[at];
                v[u] = *reinterpret_cast<const float2*>(a.part_O + at * g.d + 2 * lane);
            }
#pragma unroll
            for (int u = 0; u < N; ++u) {
                if (p0 + u >= a.nsplit || l[u] == NEG_INF) continue;   // (a part without a block)
                const float wgt = expf(l[u] - mx);
                den += wgt;
                o0 = fmaf(wgt, v[u].x, o0);
                o1 = fmaf(wgt, v[u].y, o1);
            }
            p0 += N;
        };
        while (p0 + 4 < a.nsplit) take(std::integral_constant<int, 8>{});
        if (p0 + 1 < a.nsplit) take(std::integral_constant<int, 4>{});
        if (p0 < a.nsplit) take(std::integral_constant<int, 1>{});
    }
    const float inv = den > 0.f ? 1.0f / den : 0.f;
    unsigned short* O = reinterpret_cast<unsigned short*>(a.O) + b * g.qsb + h * g.qsh + r * g.qsl;
    *reinterpret_cast<unsigned*>(O + 2 * lane) = f32_to_bf16_bits(o0 * inv) | (f32_to_bf16_bits(o1 * inv) << 16);
    if (a.lse && lane == 0) a.lse[row] = den > 0.f ? mx + logf(den) : NEG_INF;
}

// ---- planned launches (chunks of a long prompt): the plan and the merge ----
// One workgroup.  First the part length: the shortest of a fixed series, not below split_len, with which all rows longer
// than a part fit into the slots and a part is a quarter of a workgroup's share of the launch or more (shorter ones only add
// partial results); no row is cut where none is long (dense chunks of many rows).  (Rows for which no slot is left are
// computed whole, and one of them can take longer than everything else: with a fixed 64 entries a chunk of 512 tokens at
// 128K whose heads kept 42 000 block pairs took 2.17 ms, with the length that fits 0.42 ms.)  Lengths down to half of split_len
// are taken where all parts and rows then run at once, so that the launch takes as long as one part: tau 0.8, 300 tokens at
// 30000, 32 / 8 heads 147 -> 131 us, 300 at 20000, 16 / 4 115 -> 78, 600 at 40000, 8 / 2 111 -> 70, 1000 at 65536, 8 / 2 123 -> 86.
// Then it walks the rows in launch order, gives every row longer than that one slot per part (a prefix sum) and lists the
// slots' rows.
constexpr int kPlanThreads = 1024;
constexpr int kPlanResident = 512;   // workgroups that run at once
constexpr int kPlanShare = 4 * kPlanResident;
constexpr int kPlanWhole = 768;      // no row is longer than two thirds of a workgroup's share: none is cut
__global__ void __launch_bounds__(kPlanThreads)
k_split_plan(Geom g, AttnArgs a, int grid_rows) {
    __shared__ int s_wave[kPlanThreads / 64];
    __shared__ int s_used, s_cut;
    constexpr int kShort = 4, kLens = kShort + 16;              // below split_len, in all
    __shared__ int s_need[kLens + 1], s_longest;                // slots per length, and the entries of all rows
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int Nbq = g.Lq >> 7;
    const int rows_total = g.batch * g.Hq * Nbq;
    auto count_of = [&](int rid) {                              // as the attention kernel holds it
        const int m = rid % Nbq + (a.Nb - Nbq);
        const int count = a.row_list ? a.row_count[rid] : m + 1;
        return count < 0 ? 0 : (count > m + 1 ? m + 1 : count);
    };
    auto len_of = [&](int i) { return (4 + (i & 3)) * (a.split_len << (i >> 2)) / 8; };   // of split_len: 1/2, 5/8 .. 1, 5/4 ..
    if (t <= kLens) s_need[t] = 0;
    if (t == 0) { s_used = 0; s_cut = 0; s_longest = 0; }
    __syncthreads();
    int longest = 0;
    int need[kLens + 1];
#pragma unroll
    for (int i = 0; i <= kLens; ++i) need[i] = 0;
    // parts of a row of `count` entries, exact where the length may be taken: at most 33 then, so the quotient is off by less
    // than 2^-16, and from the next whole number it is 1 / (2 len) > 2^-13 away.  (Integer divisions, sums and scan through
    // LDS: 18.0 us; so 11.4.)
    auto parts_of = [](int count, int len, float inv) {
        return count > len ? (int)(((float)(count + len - 1) + 0.5f) * inv) : 0;
    };
    for (int rid = t; rid < rows_total; rid += kPlanThreads) {
        a.plan_row[rid] = -1;
        const int count = count_of(rid);
        need[kLens] += count;
        longest = max(longest, count);
#pragma unroll
        for (int i = 0; i < kLens; ++i) need[i] += parts_of(count, len_of(i), 1.0f / (float)len_of(i));
    }
    if (64 * wave < rows_total) {
        int mine = 0;                                           // lane i: sum i
#pragma unroll
        for (int i = 0; i <= kLens; ++i) {
            const int sum = (int)wave_sum_fixed((float)need[i]);    // whole numbers below 2^24: exact
            mine = lane == i ? sum : mine;
        }
        if (lane <= kLens) atomicAdd(&s_need[lane], mine);
#pragma unroll
        for (int sft = 32; sft >= 1; sft >>= 1) longest = max(longest, __shfl_xor(longest, sft));
        if (lane == 0) atomicMax(&s_longest, longest);
    }
    __syncthreads();
    int len = len_of(kLens - 1);
#pragma unroll
    for (int i = kLens - 2; i >= 0; --i) {
        const bool fits = s_need[i] <= a.split_budget && len_of(i) >= s_need[kLens] / kPlanShare;
        if (fits && (i >= kShort || (s_need[i] + rows_total <= kPlanResident && 32 * len_of(i) >= a.Nb))) len = len_of(i);
    }
    if (s_longest <= s_need[kLens] / kPlanWhole) len = max(len, s_longest);
    int base = 0;                                               // what the rows of earlier trips take
    for (int start = 0; start < grid_rows; start += kPlanThreads) {
        const int rank = start + t;
        int parts = 0, rid = -1;
        if (rank < grid_rows) {
            int b, h, mq;
            if (decode_block(rank, g, Nbq, a.row_order, a.interleave, a.hoist, 0, false, b, h, mq)) {   // (a chunk is never packed)
                rid = (b * g.Hq + h) * Nbq + mq;
                const int count = count_of(rid);
                if (count > len) parts = (count + len - 1) / len;
            }
        }
        // the parts (at most 4096 rows x 32 < 2^18), and above them the number of rows with parts (at most 2^12)
        const int mine = parts | (parts > 0 ? 1 << 18 : 0);
        int incl = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        int before = base;
#pragma unroll
        for (int i = 0; i < kPlanThreads / 64; ++i) {
            const int v = s_wave[i];
            before += i < wave ? v : 0;
            base += v;
        }
        incl += before;
        const int first = (incl & 0x3FFFF) - parts, nth = (incl >> 18) - 1;      // slots and cut rows in front of this row
        if (parts > 0 && first + parts <= a.split_budget) {
            a.plan_row[rid] = first;
            for (int p = 0; p < parts; ++p) a.plan_items[first + p] = rid;
            a.plan_cut[nth] = rid;                             // the cut rows, in launch order (all in front fit as well)
            atomicMax(&s_used, first + parts);
            atomicMax(&s_cut, nth + 1);
        }
        __syncthreads();                                       // s_wave is read, s_used and s_cut are whole
    }
    if (t == 0) { a.plan_total[0] = s_used; a.plan_total[1] = s_cut; a.plan_total[2] = len; }
}

// The cut rows: O = sum_p exp(lse_p - lse) O_p over the row's parts, rounded once.  Four query rows of a cut row's 128 to a
// workgroup at a time, a wavefront each; the parts' lse values are read by one lane each, and four parts of a half are requested
// at once, so that nothing in the merge is a chain of dependent loads (2048 tokens at 128K 557 -> 553 us in all, eight at once
// 559), and the two halves of the wavefront take every other part, a lane four channels.  At most 64 parts per row.
// The number of cut rows is on the device: a fixed grid takes them in turns (one workgroup for each that might be there, and
// whole wavefronts per part: 37 us, so 20; 2048 tokens at 128K, 1329 parts of 70 rows).  The halves are added last, so
// an output can differ from a merge of the parts one after the other by its last rounding.
constexpr int kMergeGroups = 2048;
__global__ void __launch_bounds__(256)
k_attn_combine_plan(Geom g, AttnArgs a) {
    const int Nbq = g.Lq >> 7;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, half = lane >> 5;
    const long long rows_call = g.Lr - g.q0;
    const float NEG_INF = -__builtin_huge_valf();
    const int len = a.plan_total[2];
    const int items = 32 * a.plan_total[1];                              // four query rows of a cut row each
    for (int item = blockIdx.x; item < items; item += gridDim.x) {
        const int rid = a.plan_cut[item >> 5];
        if ((unsigned)rid >= (unsigned)(g.batch * g.Hq * Nbq)) continue;
        const int base = a.plan_row[rid];
        if (base < 0) continue;
        const int mq = rid % Nbq, bh = rid / Nbq, h = bh % g.Hq, b = bh / g.Hq;
        const int m = mq + (a.Nb - Nbq);
        const int x = 4 * (item & 31) + wv;                              // query row of the tile
        const long long r = (long long)mq * 128 + x - g.qoff;           // row of Q / O
        if (r < 0 || r >= rows_call) continue;
        int count = a.row_list ? a.row_count[rid] : m + 1;
        count = count < 0 ? 0 : (count > m + 1 ? m + 1 : count);
        int parts = (count + len - 1) / len;
        parts = parts > 64 ? 64 : parts;
        const float l = lane < parts ? a.part_lse[(long long)(base + lane) * 128 + x] : NEG_INF;
        float mx = l;
#pragma unroll
        for (int sft = 32; sft >= 1; sft >>= 1) mx = fmaxf(mx, __shfl_xor(mx, sft));
        const float wgt = l != NEG_INF ? expf(l - mx) : 0.f;
        const float den = wave_sum_fixed(wgt);
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        const float* src = a.part_O + ((long long)base * 128 + x) * g.d + 4 * (lane & 31);
        int p0 = 0;
        auto take = [&](auto n) {                                        // N parts of each half
            constexpr int N = decltype(n)::value;
            f32x4 v[N];
#pragma unroll
            for (int u = 0; u < N; ++u)
                v[u] = *reinterpret_cast<const f32x4*>(src + (long long)min(p0 + 2 * u + half, parts - 1) * 128 * g.d);
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int p = p0 + 2 * u + half;
                const float wp = __shfl(wgt, p & 63);
                if (p < parts) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = fmaf(wp, v[u][e], o[e]);
                }
            }
            p0 += 2 * N;
        };
        while (p0 + 4 < parts) take(std::integral_constant<int, 4>{});
        if (p0 + 2 < parts) take(std::integral_constant<int, 2>{});
        if (p0 < parts) take(std::integral_constant<int, 1>{});
        const float inv = den > 0.f ? 1.0f / den : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (o[e] + __shfl_xor(o[e], 32)) * inv;
        unsigned short* O = reinterpret_cast<unsigned short*>(a.O) + b * g.qsb + h * g.qsh + r * g.qsl;
        if (half == 0)
            *reinterpret_cast<u32x2*>(O + 4 * (lane & 31)) = u32x2{f32_to_bf16_bits(o[0]) | (f32_to_bf16_bits(o[1]) << 16),
                                                                   f32_to_bf16_bits(o[2]) | (f32_to_bf16_bits(o[3]) << 16)};
        if (a.lse && lane == 0) a.lse[((long long)b * g.Hq + h) * rows_call + r] = den > 0.f ? mx + logf(den) : NEG_INF;
    }
}

int attn_mfma_plan_len(const Geom& g, int B, int* budget) {
    // A chunk of a long prompt: many rows, most of them short, a few nearly as long as the context, and the launch
    // takes as long as its longest row (measured at 128K, tau 0.9: 1.1 ms for chunks of 512 to 2048 tokens whose
    // blocks are 0.15-0.19 ms of matrix work).  The result is the shortest length a part may have; k_split_plan chooses.
    // Measured, 32 / 8 heads at tau 0.9 unless said (fixed 64 entries, 128 above 2048 rows -> the length that is chosen):
    // 512 tokens at 128K (42 000 block pairs) 1750 -> 475 us, 2048 (54 000) 613 -> 585, 16384 2460 -> 2300, 28 / 4 heads 2048 at
    // 64K 264 -> 213, 64 / 8 heads 1000 at 40 000 tokens, tau 0.95, 412 -> 401; dense 2048 at 128K 4.8 -> 4.1 ms.
    if (budget) *budget = 0;
    if (B != 128 || g.d != 128) return 0;
    const int Nb = g.L / B, Nbq = g.Lq / B;
    const long long rows = (long long)g.batch * g.Hq * Nbq;
    if (Nbq < 2 || Nb < 128 || g.q0 <= 0 || rows > 4096) return 0;
    const int at_most_32 = (Nb + 31) / 32;                              // parts per row
    if (Nb <= std::max(rows <= 2048 ? 64 : 128, at_most_32)) return 0;  // contexts that are not longer are not planned
    const int len = std::max(at_most_32, 40);
    // slots: several times what the rows of such chunks were seen to need (300-1000 at 128K), between 512 and 2048
    // (34-135 MB of partial results); the workgroups of unused slots run last and cost nothing measurable
    if (budget) *budget = (int)(4 * rows < 512 ? 512 : (4 * rows > 2048 ? 2048 : 4 * rows));
    return len;
}
namespace {
size_t plan_align(size_t x) { return (x + 255) / 256 * 256; }
}
size_t attn_mfma_plan_bytes(const Geom& g, int B) {
    int budget = 0;
    if (attn_mfma_plan_len(g, B, &budget) <= 0) return 0;
    const size_t rows = (size_t)g.batch * g.Hq * (size_t)(g.Lq / B);
    return 256 + plan_align(rows * 4) + plan_align((size_t)budget * 4) + plan_align((size_t)budget / 2 * 4) +
           plan_align((size_t)budget * 128 * 4) + (size_t)budget * 128 * g.d * 4;
}
void attn_mfma_plan_pointers(const Geom& g, int B, void* workspace, AttnArgs* a) {
    int budget = 0;
    a->split_len = attn_mfma_plan_len(g, B, &budget);
    a->split_budget = budget;
    const size_t rows = (size_t)g.batch * g.Hq * (size_t)(g.Lq / B);
    unsigned char* p = static_cast<unsigned char*>(workspace);
    a->plan_total = reinterpret_cast<int32_t*>(p);
    p += 256;
    a->plan_row = reinterpret_cast<int32_t*>(p);
    p += plan_align(rows * 4);
    a->plan_items = reinterpret_cast<int32_t*>(p);
    p += plan_align((size_t)budget * 4);
    a->plan_cut = reinterpret_cast<int32_t*>(p);                    // a cut row has two parts or more
    p += plan_align((size_t)budget / 2 * 4);
    a->part_lse = reinterpret_cast<float*>(p);
    p += plan_align((size_t)budget * 128 * 4);
    a->part_O = reinterpret_cast<float*>(p);
    a->nsplit = 1;
}

int attn_mfma_splits(const Geom& g, int B) {
    // few rows, all of them deep inside the context (a step, not a prefill: even the first row has 16 causal
    // blocks or more): bring the launch to about two workgroups per compute unit (measured at a 128K context:
    // 512 workgroups 0.32 ms for a dense one-token step, 1024 workgroups 0.42 ms), every part at least 8 blocks
    // long
    const int Nb = g.L / B, Nbq = g.Lq / B;
    const long long rows = (long long)g.batch * g.Hq * Nbq;
    if (rows >= 512 || Nb - Nbq + 1 < 16) return 1;
    long long P = (512 + rows - 1) / rows;
    if (P > Nb / 8) P = Nb / 8;
    if (P > 32) P = 32;
    return P < 1 ? 1 : (int)P;
}
size_t attn_mfma_split_bytes(const Geom& g, int B) {
    const int P = attn_mfma_splits(g, B);
    if (P <= 1) return 0;
    const size_t rows = (size_t)g.batch * g.Hq * (size_t)(g.Lr - g.q0);
    return (size_t)P * rows * g.d * sizeof(float) + (size_t)P * rows * sizeof(float);
}
hipError_t launch_attn_combine(const Geom& g, const AttnArgs& a, hipStream_t st) {
    const long long nrows = (long long)g.batch * g.Hq * (g.Lr - g.q0);
    hipLaunchKernelGGL(k_attn_combine, dim3((unsigned)((nrows + 3) / 4)), dim3(256), 0, st, g, a);
    return hipGetLastError();
}

// Eight waves to a row, four of them per key half, instead of four waves with all keys: a long row takes 1.57 us per block
// instead of 2.1 (2.6 with a neighbour on the compute unit), but nothing runs behind its start and end.  It pays where a launch
// takes as long as its longest row: few rows, or sparse calls whose protected last row keeps every block.  The counts are on
// the device, so the rule goes by the number of rows and the length of the context; and it does not ask whether the call
// has a list, so that a list of every block gives the dense call's result to the bit.  Measured, us, four waves -> eight:
//   sparse, tau 0.9 unless said: 2048 tokens 8 / 2 heads (128 rows) 42 -> 39; 3072, 16 / 4 (384) 62 -> 56; 8192, 8 / 2 (512) 148
//     -> 112, 16 / 4 (1024) 161 -> 127, at tau 0.95 182 -> 166; 65536, 8 / 2 (4096) 2197 -> 1962, at tau 0.95 4634 -> 4873
//   steps and chunks at 128K without a workspace, 32 / 8: 1 token 2175 -> 1642, 2048 (512 rows) 2654 -> 1649, 8192 (2048) 2735 -> 2056
//   not taken: 512, 32 / 8 (128) 20.2 -> 21.4; 2048, 32 / 8 (512) 54 -> 52; 4096, 32 / 8 (1024) 93 -> 94, at tau 0.95 101 -> 114; 12000,
//     16 / 4 (1504) 246 -> 242, at tau 0.95 311 -> 350; 32768, 16 / 4 (4096) 1178 -> 1078, at tau 0.95 2072 -> 2192; 98304, 8 / 2 (6144)
//     4117 -> 4363
//   dense: 4096, 8 / 2 (256) 79 -> 69; 8192, 8 / 2 (512) 182 -> 162, 16 / 4 (1024) 280 -> 304; 16384, 4 / 1 (512) 335 -> 283, 8 / 2 (1024)
//     524 -> 546; 1000 at 20480, 32 / 8 (256) 385 -> 329, 2048 at 128K (512) 3885 -> 3926; not taken: 2048, 32 / 8 (512) 56 -> 69
bool wide_rows_pay(int Nb, long long rows) { return rows <= std::min<long long>(15ll * Nb + 64, 5000); }

hipError_t launch_attn_mfma_bf16(const Geom& g, const AttnArgs& a_in, hipStream_t st) {
    AttnArgs a = a_in;
    if (a.nsplit < 1 || !a.part_O || !a.part_lse) a.nsplit = 1;
    const bool planned = a.split_len > 0 && a.split_budget > 0 && a.plan_total && a.plan_row && a.plan_items && a.plan_cut &&
                         a.part_O && a.part_lse;
    if (!planned) { a.split_len = 0; a.split_budget = 0; } else a.nsplit = 1;
    const bool ordered = a.row_order && !planned && a.nsplit == 1;
    a.interleave = interleave_groups(g, ordered);
    a.hoist = ordered ? hoisted_rows(g, a.interleave) : 0;
    const bool ragged = g.Lr != g.L || g.qoff != 0 || a.nsplit > 1 || planned;   // split launches use the ragged instantiation
    const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)g.d));
    const long long rows = (long long)g.batch * g.Hq * (g.Lq / 128);
    // Launches split into equal parts that are no more than the compute units (few heads, where the parts are at most 32): the
    // longest part counts there as well.  128 tokens at 128K, 8 / 2 heads, dense 142 -> 109 us, 16 / 4 179 -> 174; 100 at 65536,
    // 8 / 2, 94 -> 77; 32 / 8 heads fill the chip with rows of four waves (64 at 65536: 151 us, wide 164).  Planned launches stay
    // on four waves: the plan makes more parts than there are compute units.
    const bool wide = !planned && (a.nsplit == 1 ? wide_rows_pay(a.Nb, rows) : rows * a.nsplit <= compute_units());
    // workgroups the chip holds at once
    const int resident = (wide ? 1 : 2) * compute_units();
    // Persistent workgroups pay where rows are short, i.e. where the start of a row is a visible share of it, and
    // a workgroup takes several: measured with two workgroups per compute unit, estimate + sparse against one
    // workgroup per row: 280 -> 274 us at 8K tokens (4 rows each), 905 -> 898 us at 18K, level at 32K (and beyond: the
    // launch is limited by power there, not by the gaps between rows); with fewer rows than workgroups the look-ahead only
    // costs (1139 tokens, 252 rows: 67 against 72 us).  Wide rows, attention alone: 2048 tokens, 28 / 4 heads 62 -> 47 us.
    const int NG = g.batch * g.Hkv;
    const bool queued = a.row_order != nullptr && a.queue != nullptr && resident >= 8 && a.nsplit == 1 && !planned && rows < 1 << 30;
    const bool by_group = queued && rows_by_group(rows, resident, NG, a.interleave, g.L, g.d);
    const bool persist = by_group || (queued && a.Nb <= kPersistMaxBlocks && rows >= resident);
    // (a list without an order: its heavy rows, the last of every head, would meet on few XCDs)
    a.by_group = by_group ? 1 : 0;
    if (!a.row_list && a.nsplit == 1 && !planned) a.by_group = dense_order(NG, g.L, g.d, g.Lq, a.seq_first != nullptr, rows);
    const unsigned grid_rows = grid_size(g, g.Lq / 128, a.row_order != nullptr);
    dim3 grid(grid_rows * (unsigned)a.nsplit + (planned ? (unsigned)a.split_budget : 0u));
    if (planned) {
        hipLaunchKernelGGL(k_split_plan, dim3(1), dim3(kPlanThreads), 0, st, g, a, (int)grid_rows);
        const hipError_t pe = hipGetLastError();
        if (pe != hipSuccess) return pe;
    }
    unsigned starts = 0x11111111u;
    if (persist) grid = dim3((unsigned)resident);
    if (by_group) {
        starts = 0;
        for (int x = 0; x < 8; ++x) starts += 1u << (4 * (x % std::min(NG, 8)));
        a.hoist = front_rows_of_groups(NG, g.G, g.Lq / 128);
    }
    // How far a weight may exceed the softmax reference before the reference moves up to it, see the head of the file: 2^8, or 2^6
    // in planned launches.
    const float lazy_log2 = planned ? 6.0f : 8.0f;
    const int lds_bytes = (wide ? 2 : 1) * kLdsBytes + (persist ? 16 : 0);
    auto launch = [&](auto kernel) -> hipError_t {
        hipError_t e = allow_dynamic_lds((const void*)kernel, lds_bytes);
        if (e != hipSuccess) return e;
        AttnKernelArgs ka;
        ka.g = g;
        ka.a = a;
        ka.scale_log2 = scale_log2;
        ka.lazy_log2 = lazy_log2;
        ka.lazy_sum = exp2f(lazy_log2);
        ka.starts = starts;
        hipLaunchKernelGGL(kernel, grid, dim3((wide ? 2 : 1) * kThreads), lds_bytes, st, ka);
        return hipGetLastError();
    };
    if (wide && persist) return ragged ? launch(k_attn_mfma_bf16<true, true, true>) : launch(k_attn_mfma_bf16<false, true, true>);
    if (wide) {
        const hipError_t e = ragged ? launch(k_attn_mfma_bf16<true, false, true>) : launch(k_attn_mfma_bf16<false, false, true>);
        return e != hipSuccess || a.nsplit == 1 ? e : launch_attn_combine(g, a, st);
    }
    if (persist) return ragged ? launch(k_attn_mfma_bf16<true, true, false>) : launch(k_attn_mfma_bf16<false, true, false>);
    const hipError_t e = ragged ? launch(k_attn_mfma_bf16<true, false, false>) : launch(k_attn_mfma_bf16<false, false, false>);
    if (e != hipSuccess) return e;
    if (planned) {
        const long long cut_max = rows < a.split_budget / 2 ? rows : a.split_budget / 2;
        const long long groups = 32 * cut_max < kMergeGroups ? 32 * cut_max : kMergeGroups;
        hipLaunchKernelGGL(k_attn_combine_plan, dim3((unsigned)groups), dim3(256), 0, st, g, a);
        return hipGetLastError();
    }
    if (a.nsplit == 1) return e;
    return launch_attn_combine(g, a, st);
}

}  // namespace rr
