// Scheduling hint for the sparse attention launch: per (batch, KV head) the rows (hl, m) of its G
// query heads in the order their workgroups should start.
//
// Balance.  Workgroups are handed to the XCDs round-robin in launch order and a workgroup cannot start
// before the one launched ahead of it: rows of very different length next to each other (Top-tau
// keeps anything from a handful of blocks to all of them, Sec. 3.3) leave compute units idle, rows of
// equal length side by side do not.  Rows are therefore sorted by count class (count / 8), heaviest
// class first.
// Locality.  Inside a class rows go by descending query block, the G heads of a query block together:
// such neighbours select many of the same key blocks and walk them at the same pace.  Within every
// run of 8 G sorted rows the launch ranks are transposed, so that G consecutive sorted rows get ranks 8
// apart and meet in the L2 of one XCD.  The order is a pure function of the counts (deterministic).
//
// One workgroup per (batch, KV head) counts the rows of every class and then places the rows in the order of (descending
// query block, head): a row's rank is its class's start, the rows of its class in front of its wavefront, and those in
// front of its lane.  G * Nb <= 32768 rows (the caller checks).  What bounds it is the chain of its barriers; a bitonic
// sort of (class, row) keys, the form before, had log^2 as many: 2177 rows 31 -> 11 us, 512 rows
// 9.5 -> 4.8, 4096 rows 33 -> 17.
#include "rr_common.hpp"

namespace rr {

namespace {

constexpr int kCountShift = 3;      // rows whose counts differ by less than 8 blocks form one class
constexpr int kMaxClasses = 4096;   // (beyond 32K blocks classes are wider)

template <int kSortThreads>                         // at least RR_QUEUE_WORDS
__global__ void __launch_bounds__(kSortThreads)
k_row_order(Geom g, int Nb, int shift, const int32_t* __restrict__ row_count, int32_t* __restrict__ row_order,
            int32_t* __restrict__ queue) {
    __shared__ int start[kMaxClasses];                  // rows of a class, then where its next row goes
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int kv = blockIdx.x, b = blockIdx.y;
    // the row counters of the attention launch that will follow this order start from zero
    if (queue && kv == 0 && b == 0 && t < RR_QUEUE_WORDS) queue[t] = 0;
    const int Nbq = g.Lq / (g.L / Nb);                  // rows per head (chunked prefill: the last Nbq query blocks)
    const int N = g.G * Nbq;
    const int classes = (Nb >> shift) + 1;              // at most kMaxClasses (the host)
    const int32_t* cnt = row_count + ((long long)b * g.Hq + (long long)kv * g.G) * Nbq;   // G heads, contiguous
    for (int c = t; c < classes; c += kSortThreads) start[c] = 0;
    __syncthreads();
    auto class_of = [&](int f) {                        // f = (Nbq-1-m) G + hl: m descending, then head
        const int mr = f / g.G, hl = f - mr * g.G;
        int c = cnt[hl * Nbq + (Nbq - 1 - mr)];
        c = c < 0 ? 0 : (c > Nb ? Nb : c);
        return (Nb - c) >> shift;
    };
    for (int f = t; f < N; f += kSortThreads) atomicAdd(&start[class_of(f)], 1);
    __syncthreads();
    if (wv == 0) {                                      // exclusive prefix sum over the classes
        int run = 0;
        for (int c0 = 0; c0 < classes; c0 += 64) {
            const int v = c0 + lane < classes ? start[c0 + lane] : 0;
            int incl = v;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int up = __shfl_up(incl, o);
                incl += lane >= o ? up : 0;
            }
            if (c0 + lane < classes) start[c0 + lane] = run + incl - v;
            run += __shfl(incl, 63);
        }
    }
    __syncthreads();
    int32_t* out = row_order + ((long long)b * g.Hkv + kv) * N;
    // Rows that are neighbours in the sorted sequence (same count class, same or adjacent query block, the
    // G heads of one KV head) share many key blocks and walk them at the same pace.  Workgroups go to the
    // XCDs round-robin in launch order, so within every run of 8 G sorted rows the launch order is
    // transposed: G consecutive sorted rows get ranks 8 apart and meet in the L2 of one XCD.
    const int C = g.G;
    const int full = N / (8 * C) * (8 * C);
    for (int f0 = 0; f0 < N; f0 += kSortThreads) {
        const int f = f0 + t;
        const bool in = f < N;
        const int c = in ? class_of(f) : 0;
        unsigned long long same = __ballot(in);         // lanes of this wavefront with a row of the same class
        for (int bit = 1; bit < classes; bit <<= 1) {
            const unsigned long long set = __ballot((c & bit) != 0);
            same &= (c & bit) ? set : ~set;
        }
        int pos = 0;
        const int waves = min(kSortThreads, N - f0 + 63) >> 6;      // wavefronts with rows take their places in turn
        for (int w = 0; w < waves; ++w) {
            if (wv == w && in && lane == __ffsll(same) - 1) pos = atomicAdd(&start[c], __popcll(same));
            __syncthreads();
        }
        const int i = __shfl(pos, in ? __ffsll(same) - 1 : lane) + __popcll(same & ((1ull << lane) - 1ull));
        if (in) {
            const int mr = f / g.G, hl = f - mr * g.G;
            int rank = i;
            if (C > 1 && i < full) {
                const int base = i / (8 * C) * (8 * C), w = i - base;
                rank = base + 8 * (w % C) + w / C;
            }
            out[rank] = hl * Nbq + (Nbq - 1 - mr);
        }
    }
}

// dense 0/1 rows -> count and ascending list, one wave per (batch, head, row); entries above the
// diagonal are ignored.  Lanes scan 64 columns at a time, the rank of a set column is the count of set
// columns before it (ballot + popcount).
__global__ void __launch_bounds__(256)
k_mask_from_dense(long long rows, int Nb, int Nbq, const uint8_t* __restrict__ dense, int32_t* __restrict__ row_count,
                  int32_t* __restrict__ row_list) {
    const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int lane = threadIdx.x & 63;
    const int m = (Nb - Nbq) + (int)(row % Nbq);
    const uint8_t* src = dense + row * Nb;
    int32_t* dst = row_list + row * Nb;
    int count = 0;
    for (int n0 = 0; n0 <= m; n0 += 64) {
        const int n = n0 + lane;
        const bool set = n <= m && src[n] != 0;
        const unsigned long long bal = __ballot(set);
        if (set) dst[count + __popcll(bal & ((1ull << lane) - 1ull))] = n;
        count += __popcll(bal);
    }
    if (lane == 0) row_count[row] = count;
}

}  // namespace

hipError_t launch_mask_from_dense(const Geom& g, int Nb, const uint8_t* dense, int32_t* row_count, int32_t* row_list,
                                  hipStream_t st) {
    const int Nbq = g.Lq / (g.L / Nb);
    const long long rows = (long long)g.batch * g.Hq * Nbq;
    hipLaunchKernelGGL(k_mask_from_dense, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, rows, Nb, Nbq, dense,
                       row_count, row_list);
    return hipGetLastError();
}

int row_order_shift(int Nb) {
    int shift = kCountShift;
    while ((Nb >> shift) + 1 > kMaxClasses) ++shift;
    return shift;
}

hipError_t launch_row_order(const Geom& g, int Nb, const int32_t* row_count, int32_t* row_order, int32_t* queue,
                            hipStream_t st) {
    const int N = g.G * (g.Lq / (g.L / Nb));
    if (N > kMaxOrderedRows) return hipErrorInvalidValue;
    const dim3 grid(g.Hkv, g.batch);
    const int shift = row_order_shift(Nb);
    // No more wavefronts than rows fill: they wait for each other at every barrier.  Estimate and attention with 1024
    // threads / these, us: fp32, 4096 tokens, 8 / 2 heads (256 rows) 188.9 / 187.0, bf16, 2048, 32 / 8 (64) 65.5 / 64.8,
    // 8153, 16 / 4 of 64 (512) 181.3 / 180.0.
    auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, st, g, Nb, shift, row_count, row_order, queue);
    };
    if (N <= 256) launch(k_row_order<256>, 256);
    else if (N <= 512) launch(k_row_order<512>, 512);
    else launch(k_row_order<1024>, 1024);
    return hipGetLastError();
}

}  // namespace rr
