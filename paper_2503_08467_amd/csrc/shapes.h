// Which kernel and which tile a call takes, from the sizes that the host knows: plain functions
// (no HIP), so that they can be checked by themselves.  `cus` is the device's number of CUs; the
// figures beside the rules were measured at 256.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace moe {

// ---- Step 1

// Streaming the K chunks through LDS (route_lds_kernel) pays where the gate is large: 64 experts,
// 32768 tokens 20.4 us against 44.5 for route_kernel, 128 experts, 30000 tokens 23.5 against 39.8,
// 64 tokens 9.6 against 14.4.  (17 to 32 experts would gain with many tokens and lose with few,
// and which of the two a call takes must not depend on its tokens: a token's logits have the same
// bits in any batch.)
inline bool route_in_lds(bool bf16, int h, int E) { return bf16 && h % 64 == 0 && E > 32; }

// route_kernel: waves of a workgroup, and K steps of 64 bytes in the longest of their runs.
inline int route_waves(int E) { return E <= 64 ? 8 : 4; }
inline int route_run(bool bf16, int h, int E) {
    const int steps = (h * (bf16 ? 2 : 4) + 63) / 64, w = route_waves(E);
    return (steps + w - 1) / w;
}

// Whether one routing workgroup covers the whole batch, so that it also groups the assignments
// (k <= 8 picks are kept in registers).  The launch that this saves is worth about 1.3 us; a
// second block of 16 tokens or more in one workgroup, instead of a workgroup each, costs in
// proportion to a row's bytes.  One launch / two (us):
// 64 tokens, 8 experts, bf16: h = 512 7.3 / 8.9, 1024 9.3 / 9.0, 4096 21.6 / 12.5; 32 experts,
//   fp32: h = 512 12.6 / 10.2, 4096 54 / 31; 64 experts, h = 1000 13.3 / 12.6;
// 32 tokens: 8 experts, bf16 h = 1536 8.3 / 9.0, 2048 10.1 / 9.1; fp32 h = 768 8.7 / 8.9, 1024
//   10.4 / 9.2; 32 experts, bf16 h = 4096 19.8 / 20.4, 8192 33 / 30; fp32 h = 2048 21.0 / 20.9,
//   4096 35 / 31; 60 experts, bf16 h = 2056 15.3 / 16.6; 128 experts, h = 1000 15.1 / 16.4;
// fp32 with more than 32 experts, at 17 tokens: 60 experts, h = 2056 32.1 / 32.1 (its matrix rate).
inline bool route_groups(bool bf16, int64_t T, int h, int E, int k) {
    if (T < 1 || T > 64 || k > 8) return false;
    if (T <= 16 || route_in_lds(bf16, h, E)) return true;
    const int64_t row = static_cast<int64_t>(h) * (bf16 ? 2 : 4);
    if (T > 32) return E <= (bf16 ? 64 : 32) && row <= 1024;
    return E <= 32 ? row <= (E <= 16 ? 3072 : 8192) : bf16 && E <= 128;
}

// Blocks of 16 tokens per workgroup of route_kernel.  A batch that is grouped in the same launch
// (route_groups) takes as many as it has.  Otherwise one while that fits the CUs in one round
// (2500 tokens, 8 experts, h = 4096 10.1 us, 17.4 with two) and the gate is small; two beyond (8192
// tokens, 4 experts, h = 1024 9.7 with one, 7.8; 8192 tokens, 256 experts, h = 1000 52 with one, 35)
// or where re-reading the gate per workgroup costs more (300 tokens, 60 experts 10.4 and 9.7); four
// for 17 to 32 experts from two such rounds on (30000 tokens, h = 768 33.2 with two, 27.5; 8192
// tokens 16.3, 17.5).
inline int route_blocks(int64_t T, int E, bool group, int cus) {
    if (T <= 16) return 1;
    if (group) return T > 32 ? 4 : 2;
    const int64_t round = 16 * static_cast<int64_t>(cus);
    if (E > 16 && E <= 32 && T >= 4 * round) return 4;
    return T > round || (E > 32 && E <= 128) ? 2 : 1;
}

// K steps per stage of loads: a stage that runs past the end of a wave's run loads its last step
// again, so short runs want short stages.  At most 16 experts: with one block 4, or 6 where that
// loads fewer steps (512 tokens, fp32, h = 768, runs of 6 10.9 us at 4, 10.0 at 6; 8, which every run
// had, 10.7, and 10.5 against 9.1 at h = 1024 in bf16, runs of 4); with two 2, or 3 likewise (8192
// tokens, h = 1024, runs of 4 17.1 at 2, 18.3 at 3; 30000 tokens, h = 768, runs of 3 26.5 and 24.3).
// 17 to 32 experts: with one block 2 (512 tokens, h = 512 9.2, 10.3 at 5; h = 4096 18.7 and 21.5) but
// for runs of 5, one stage of 5 (h = 1280 12.2 at 2, 11.7); with more blocks 1 (12000 tokens, h = 768
// 21.5, 23.3 at 2).  Larger gates: what the registers hold.
inline int route_stage(int E, int blocks, int run) {
    const auto pick = [run](int small, int large) {
        return (run + large - 1) / large * large < (run + small - 1) / small * small ? large : small;
    };
    if (E <= 16) return blocks == 1 ? pick(4, 6) : blocks == 2 ? pick(2, 3) : 2;
    if (E <= 32) return blocks > 1 ? 1 : run == 5 ? 5 : 2;
    return E <= 64 && blocks == 1 ? 3 : 1;
}

}  // namespace moe
