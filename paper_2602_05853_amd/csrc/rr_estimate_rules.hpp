// Rules of the estimate's launches in plain C++ (HIP compiles constexpr functions for host and device), so that they can be checked
// without a GPU.
#pragma once

namespace rr {

// Whether a workgroup of the generic estimate has eight waves instead of four: `workgroups` of the launch, each with R
// sampled queries of `heads` heads against up to Nb key blocks, d channels, and with lds bytes of LDS.
// With one workgroup to a compute unit, by their number or their LDS, what bounds a launch is the chain of score tiles of a
// wave (11 of the 21 us of the last row's workgroup for 4096 tokens, fp32).  With up to two the units have two waves to a
// SIMD already: eight to a workgroup still pay where all of it is short, or for a single prompt (its heavy rows meet light
// ones on a unit; those of several prompts meet each other) of narrow heads or few workgroups beyond the first round.  Up
// to 256 blocks, whose masses the first four waves sum in the same order.
// The whole estimate, us, four waves / eight, 280 shapes of random sizes with 40 to 800 workgroups, by their number:
//   up to 256: 0.715 to 0.98 of the time, level on rows of ten blocks; 4096 tokens, fp32, 8 / 2 heads of 128 (256)
//     192.2 / 188.7 with attention
//   257 to 512, taken: bf16, 6 / 3 of 96 (282) 25.1 / 22.8, fp32, 2 / 1 of 64, R = 32 (500) 224 / 210, 4 / 2 of 96 (312)
//     42.4 / 40.0, two prompts, 2 / 2 of 24 (336) 22.7 / 19.6; with 84 KB, 2 / 1 of 128, R = 32 (500) 358 / 267
//   not taken: fp32, two prompts, 2 / 1 of 128 (500) 79.7 / 85.8, of 64 (500) 50.1 / 51.8, 3 / 1 of 136 (381) 62.6 / 65.3;
//     bf16, 4 / 2 of 80 (508) 52.5 / 54.9, two prompts, 1 / 1 of 136 (436) 361 / 442
//   more than 512: 0.86 to 1.13; 8153 tokens, 16 / 4 of 64 (1024), with attention, 180.6 / 185.4
// In the mean 0.930 of four waves' time, at worst 1.02 (rows of ten blocks, 17.9 / 18.2); all up to 512 workgroups 0.930
// and 1.22.
constexpr bool eight_waves_pay(long long workgroups, int batch, int Nb, int R, int heads, int d, unsigned lds) {
    const long long tiles = (long long)Nb * R * ((R * heads + 15) / 16) * d;       // of the longest row, times 16 x 32
    const bool is_short = workgroups * tiles <= 22000000;
    const bool alone = workgroups <= 256 || lds > 80 * 1024;                        // one to a compute unit at a time
    return Nb <= 256 && workgroups <= 512 && (alone || is_short || (batch == 1 && (d <= 64 || workgroups <= 352)));
}

}  // namespace rr
