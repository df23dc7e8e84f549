// Which kernel and which tile a call takes, from the sizes that the host knows: plain functions
// (no HIP), so that they can be checked by themselves.  `cus` is the device's number of CUs; the
// figures beside the rules were measured at 256.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

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

// ---- Step 4
//
// A: the call's row bound; E: the experts of the launch; K, N: the product's sizes.

inline int64_t tiles_of(int64_t n, int64_t d) { return (n + d - 1) / d; }

// Row tiles of bm rows that A rows of E experts can have at most.
inline int64_t row_tile_bound(int64_t A, int E, int bm) { return std::min<int64_t>(tiles_of(A, bm) + E, A); }

// Decode-sized calls, whose second product stays in fp32 sums that the combine reads
// (moe_expert_ffn_shard_gather_combine): at most 512 bf16 or 1024 fp32 rows, and a packed inner
// width fp (a multiple of 128) of at least 512 or 1024.
inline bool hands_over_sums(int64_t A, int64_t fp, bool bf16) {
    return bf16 ? A <= 512 && fp >= 512 : A <= 1024 && fp >= 1024;
}

// K parts of the second product: four where its fp32 form does not stream and hands_over_sums, so
// that few row tiles with a long K loop each spread their weight reads over more workgroups; else
// whole sums.
inline int down_parts(int64_t A, int64_t fp, bool bf16, bool stream) {
    return !bf16 && !stream && hands_over_sums(A, fp, bf16) ? 4 : 1;
}

// Bytes of fp32 sums that the workspace reserves past H for a bound of A rows: 4 x rows x h floats
// of fp32 calls (down_parts), up to 8 x 256 of bf16 ones (an earlier form split their K; the size is
// part of the ABI).  The most that any call with at most A rows has, so that a workspace sized for a
// bound also serves every smaller call.
inline size_t down_partial_bytes(int64_t A, int64_t h, int64_t fp, bool bf16) {
    const auto parts = [&](int64_t a) -> int64_t {
        if (!hands_over_sums(a, fp, bf16)) return 0;
        return !bf16 ? 4 : std::min<int64_t>(a <= 256 ? 8 : 4, fp >= 2048 && fp % 256 == 0 ? 8 : fp >= 1024 ? 4 : 2);
    };
    int64_t most = 0;
    for (int64_t end : {int64_t(256), int64_t(512), int64_t(1024)})
        most = std::max(most, parts(std::min(A, end)) * std::min(A, end));
    return static_cast<size_t>(most) * static_cast<size_t>(h) * 4u;
}

// Weight rows per workgroup of gemm_stream (SwiGLU: of both matrices together): as many of 64, 32, 16
// as still give every CU two workgroups (one from 48 rows on, where narrow ones re-read the
// activations too often: 1 expert, 64 rows 10.2 / 8.0 us at 32, 8.4 / 7.2 at 64; 8 experts, 4 fp32 rows
// 12.9 at 32, 10.9 at 16).
inline int stream_width(int64_t A, int E, int64_t N, bool swiglu, int cus) {
    const int64_t tiles = std::min<int64_t>(A, E + A / 16), want = (A < 48 ? 2 : 1) * static_cast<int64_t>(cus);
    int nc = 64;
    while (nc > (swiglu ? 32 : 16) && tiles * tiles_of(N, swiglu ? nc / 2 : nc) < want) nc /= 2;
    return nc;
}

// Blocks of 16 activation rows per workgroup of gemm_stream (of 64 weight rows; narrower ones take
// one) that suit a call's rows per expert: two
// above 8 (8 experts, 256 rows 77 / 35 -> 68 / 30 us; 64 experts, 64 rows 17.0 -> 18.4 us would lose);
// three where the experts' rows, with the spread of an even routing, need fewer tiles of 48 than of 32
// (512 rows: 16 experts, 1024 x 4096 82 -> 69 us, 8 experts 69 -> 57; but 24 rows each 64 -> 66, 96 rows
// 45 -> 49).
inline int stream_blocks(int64_t A, int E, bool bf16) {
    if (!bf16 || A <= 8 * static_cast<int64_t>(E)) return 1;
    const double rows = static_cast<double>(A) / E, most = rows + 1.3 * std::sqrt(rows);
    return E >= 4 && rows <= 72 && std::ceil(most / 48) < std::ceil(most / 32) ? 3 : 2;
}

// The same for a launch of n_tiles column tiles of 64: three only where two would give the CUs more
// than 1.2 workgroups each (8 experts, 1024 x 1024, the layer: 256 rows 22.9 us at two, 24.5 at three;
// 512 rows 29.1 and 24.5).
inline int stream_launch_blocks(int64_t A, int E, int64_t n_tiles, bool bf16, int cus) {
    const int blocks = stream_blocks(A, E, bf16);
    return blocks == 3 && (static_cast<double>(A) / 32 + 0.5 * E) * static_cast<double>(n_tiles) <= 1.2 * cus ? 2 : blocks;
}

// Which calls stream their weights (gemm_stream), from the call's sizes: the same answer for every
// launch path of a call, since the waves' K parts make its sums round differently.
//
// bf16: a streaming call reads an expert's W bytes of weights once per row tile, the first time from
// HBM, again from L2 at about 10 TB/s; the tiled kernels read them once and take the longer of that
// and of their K loops, 9 ns per element of h + fp.  So it streams where the re-reads (of half a tile
// more per expert than its rows fill) stay below what the K loops take longer than HBM.  The tiled
// kernels' row-major form (h not a multiple of 32) reads its weights more slowly.  Measured (us, the
// expert step, streamed / tiled): 1 expert (4096 x 3584 SwiGLU) 128 rows 56 / 85, 256 94 / 86, 512 153 / 90;
//   (2048 x 2048) 512 rows 37 / 45, 768 52 / 45; 4 experts (4096 x 1792 SwiGLU) 192 rows 64 / 76, 256 80 /
//   76; 8 experts (4096 x 3584 SwiGLU) 64 rows 136 / 129, 192 148 / 131, 512 244 / 138; (2048 x 2048) 384
//   rows 50 / 61, 512 64 / 61; 24 experts (1032 x 4096) 512 rows 110 / 127; 64 experts (1024 x 4096) 1000
//   rows 213 / 200.  With more than 512 rows, only up to 16 an expert.
// fp32: 8 experts (768 x 3072, up / down + split sum, tiled against streamed) 4 rows 22 / 19 + 4
//   against 11 / 11, 64 rows 29 / 27 + 5 against 26 / 28, 128 rows 29 / 27 + 4 against 33 / 41 (its
//   matrix rate is a sixteenth of bf16's); only where the tiled kernel's up-projection has at most
//   one 128-column tile per CU: with more, its 128-byte pieces of a row stream the weights faster
//   (layers of 24 experts 3456 x 488 167 -> 136, 64 experts 2624 x 168 203 -> 173, but 96 experts 832 x
//   1216 112 -> 136, 64 experts 640 x 2564 209 -> 253).
inline bool stream_rows(int64_t A, int E, int64_t h, int64_t fp, bool swiglu, bool bf16, int cus) {
    if (!bf16) return (A <= 64 || A <= 8 * static_cast<int64_t>(E)) && std::min<int64_t>(A, E) * (fp / 128) <= cus;
    if (A > 512 && A > 16 * static_cast<int64_t>(E)) return false;
    const double weights = 2.0 * (swiglu ? 3 : 2) * static_cast<double>(h) * static_cast<double>(fp);
    const double experts = static_cast<double>(std::min<int64_t>(A, E));
    const double tile = 16.0 * std::max(2, stream_blocks(A, E, true));
    const double again = std::max(static_cast<double>(A) / tile - experts / 2, 0.0) * weights;
    const double first = (h % 32 == 0 ? 1.2 : 0.8) * experts * weights;
    return again <= std::max(85e3 * static_cast<double>(h + fp) - first, 0.0);
}

// The tiled bf16 launches: activation rows x weight rows of a tile.
enum GemmShape {
    kTurns256x256,  // gemm_turns
    kPairs128x256,  // gemm_up_pairs
    kTile64x128,    // gemm_bf16_lds, as the rest
    kTile64x256,
    kTile128x128,
    kTile128x256,
    kTile128x384,
};

// Tiles of 256 rows that A rows of E experts take in all but unlikely routings: the experts' last
// tiles are half full on average, two standard deviations more at most; with even routing all alike.
inline int64_t most_tiles_256(int64_t A, int E) {
    const double most = static_cast<double>(A - 1) / 256 + 0.5 * E + std::min(0.5 * E, std::sqrt(E / 3.0));
    return std::max(static_cast<int64_t>(most), E * tiles_of(A, 256 * static_cast<int64_t>(E)));
}

// Expected rounds of 256 x 256 tiles over the CUs: half an empty row tile per expert.
inline double turns_rounds(int64_t A, int E, int64_t n_tiles, int cus) {
    return (static_cast<double>(A) / 256 + 0.5 * E) * static_cast<double>(n_tiles) / cus;
}

// Which launches take gemm_turns.  Measured over A = 768 .. 65536 rows, 1 .. 64 experts,
// K = 512 .. 4096 (us, the 128 x 256 tiles against 256 x 256):
// down-projection: K = 4096 545 / 491 (1024 rows per expert), 302 / 288 (512), 213 / 210 (256);
//   K = 2816 67 / 64 (188); K = 1792 140 / 138; but K = 1024 28 / 27 (128), K = 512 37 / 44 (512):
//   a short K loop does not pay for its fill and the single workgroup's exposed epilogue; and where
//   the 128 x 256 tiles have a CU each they win (16 experts, 1024 x 4096, 6144 rows 158 / 168 the
//   step, but 8192 rows 204 / 189; 8 experts, 4096 x 3584, 1536 rows 210 / 222, but 4 experts, 2048
//   rows 237 / 210), as they do where they fit one round of two a CU and the 256 x 256 tiles may not
//   fit theirs (8 experts, 3072 x 2816, 4674 rows the step 198 / 288, skewed 199 / 228; 32 experts, 768
//   x 3072, 18538 rows 240 / 282; where those just fit, 64 experts, 768 x 3584, 259 / 240);
// up-projection: K = 4096 941 / 799, 369 / 307, 262 / 219 and, where they surely fit one round of the
//   CUs, 141 / 124; just over one round 137 / 173 (3 experts, 6144 x 2816 SwiGLU, 2429 rows the step 284 /
//   405, 16 experts, 4096 x 1408, 3847 rows, skewed, 220 / 302, even routing 221 / 214); K = 2048 419 / 378
//   over many rounds, a tie below; K = 1024 702 / 708.
inline bool turns_rows(int64_t A, int E) { return A >= 192 * static_cast<int64_t>(E); }
inline bool turns_down(int64_t A, int E, int K) { return K >= 1536 && turns_rows(A, E); }
inline bool turns_up(int64_t A, int E, int K, int64_t n_tiles, int cus) {
    if (K % 32 != 0 || K < 1536 || !turns_rows(A, E)) return false;
    const double rounds = turns_rounds(A, E, n_tiles, cus);
    if (rounds >= 4 || K < 3072) return rounds >= 4;
    return rounds >= 1.6 || (rounds >= 0.75 && most_tiles_256(A, E) * n_tiles <= cus);
}

// Tile shape otherwise: 128 activation rows x 256 weight rows, 32-wide K steps, three stages (two in
// flight) in 72 KiB of LDS, so that two workgroups share a CU and one's epilogue and pipeline fill
// overlap the other's MFMAs.  The up-projection takes its activation rows in 128-byte pieces when
// K allows it (gemm_up_pairs).  Its weights are K-blocked when K = h is a multiple of 32; otherwise
// they are row-major and the kernel's RM form reads them, in the same shapes (1531 tokens, 24 experts,
// h = 776, f = 1365: 34.5 us, 49.7 through a register-staged kernel).  The down-projection's K is fp,
// always a multiple of 128.
//
// Few tiles leave CUs idle and few bytes in flight, so such calls take smaller ones.  Measured
// (us, up / down; each output element's K sum is the same in any shape):
// - thin experts, 64 x 256: 64 experts (1024 x 1024) 2000 rows 34 / 35 -> 30 / 30; and where one row tile
//   each gives every CU at most one 128-column tile, 64 x 128 up and 128 x 128 down: 32 experts (1024 x
//   4096) 1024 rows the layer 126 -> 111; 16 experts (2048 x 2048) 512 rows 81 -> 70; with more columns
//   than that 64 experts (768 x 768) 1536 rows 45 -> 53;
// - at most 5/8 of a 128 x 256 tile per CU, 128 x 128 in four stages, two workgroups a CU: 16
//   experts (1408 x 1024) 2000 rows 34 / 27 -> 25 / 19; 8 experts (3072 x 384 SwiGLU) 4000 rows up
//   65 -> 39; 24 experts (776 x 1365) 3062 rows down 33 -> 22; at 3/4 of a tile 31 -> 34, 25 -> 28;
// - at most 1/4, 64 x 128 for the up-projection: 4 experts (1728 x 1520) 823 rows 40 -> 18 (24 at
//   128 x 128).

// Experts whose rows fit one tile of 64: at most 40 on average, or 48 where the CUs' last round has
// room for a few second tiles.  An even routing's largest expert passes 64 rows from about 44 on, and
// where the tiles fill whole rounds its second row tile costs most of another (64 experts, 1024 x
// 1024, 3000 rows 62 -> 81 us the step; 64 experts, 1024 x 4096 208 -> 259; with room 768 x 768 43 -> 44).
inline bool thin_experts(int64_t A, int E, int64_t n_tiles, int cus) {
    if (A <= 40 * static_cast<int64_t>(E)) return true;
    const int64_t last = E * n_tiles % cus;
    return A <= 48 * static_cast<int64_t>(E) && last > 0 && last + 4 * n_tiles <= cus;
}

// Tiles of 128 rows with half an empty row tile per expert.
inline double expected_tiles(int64_t A, int E, int64_t n_tiles) {
    return (static_cast<double>(A) / 128 + 0.5 * E) * static_cast<double>(n_tiles);
}

inline GemmShape up_shape(int64_t A, int E, int K, int N, bool swiglu, int cus) {
    const int64_t n_tiles = tiles_of(N, swiglu ? 128 : 256);
    if (turns_up(A, E, K, n_tiles, cus)) return kTurns256x256;
    if (thin_experts(A, E, n_tiles, cus)) return E * tiles_of(N, swiglu ? 64 : 128) <= cus ? kTile64x128 : kTile64x256;
    const double tiles = expected_tiles(A, E, n_tiles);
    if (4 * tiles <= cus) return kTile64x128;
    if (8 * tiles <= 5 * cus) return kTile128x128;
    return K % 64 == 0 ? kPairs128x256 : kTile128x256;
}

// When the down-projection's tiles fit on the CUs in one round even 384 columns wide, and those
// waste no more columns than 256-wide ones, it runs 128 x 384 tiles, one workgroup per CU with
// 96 KiB of stages: every tile then streams its weights with more bytes in flight instead of a
// third of the CUs taking a second tile (64 experts, 3072 x 768, 8192 rows 108 -> 89; 1024 columns
// in three would lose: 26 -> 30).  That workgroup has 8 waves (2 x 4, each 64 x 96), two per SIMD, so
// that one wave's LDS reads, loads and barrier waits overlap the other's MFMAs.  With a short K the
// wasted columns cost less than the second tiles do (16 experts, 1024 x 1024, 8192 rows the step 79 ->
// 72; 8 experts, 2048 x 1408, 4096 rows 113 -> 103; but K = 2048 16 experts, 3072 rows 99 -> 106).
inline GemmShape down_shape(int64_t A, int E, int K, int N, int cus) {
    const int64_t n256 = tiles_of(N, 256), n384 = tiles_of(N, 384), row_tiles = row_tile_bound(A, E, 128);
    if (thin_experts(A, E, n256, cus)) return E * tiles_of(N, 128) <= cus ? kTile128x128 : kTile64x256;
    if (8 * expected_tiles(A, E, n256) <= 5 * cus) return kTile128x128;
    const bool fits_384 = row_tiles * n384 <= cus && (n384 * 384 <= n256 * 256 || (K < 1536 && row_tiles * n256 > cus));
    // 32 experts (1568 x 640), 9542 rows: the layer 101 us at 384 columns, 105 in turns; from
    // 375 rows per expert turns win there too (48.6 -> 45.2)
    const double tiles = expected_tiles(A, E, n256);
    if (turns_down(A, E, K) && tiles > cus && !(tiles <= 2.0 * cus && most_tiles_256(A, E) * n256 > cus) &&
        !(fits_384 && A < 320 * static_cast<int64_t>(E)))
        return kTurns256x256;
    return fits_384 ? kTile128x384 : kTile128x256;
}

}  // namespace moe
