// Step 4 of the layer: this device's shard of every expert on the rows routed to it, as a
// grouped GEMM over variable-length expert segments -- one launch per matmul, whatever
// the number of experts.
//
//   GEMM1   H[p, n] = act(x_perm[p] . W1^T[e][n])       (SwiGLU: silu(.W1) * (.W3))
//   GEMM2   y_perm[p, c] = H[p] . W2^T[e][c]
//
// Each workgroup first turns offsets[] into a per-expert prefix of row tiles, then maps
// linear tile ids to (expert, row tile, column tile).  The grid is persistent (sized from
// the host-known bound A_max, at most as many workgroups per CU as LDS allows, a multiple
// of the 8 XCDs), so the counts are never read back to the host.
//
// bf16, many rows per expert (gemm_bf16_lds, gemm_up_pairs, gemm_turns): tiles of 64 to 256
// rows, v_mfma_f32_32x32x16_bf16 with fp32 accumulation.  Weights and H are stored K-blocked
// (blocks of 32 K values, all rows side by side), so every stage of 32 K values of a run of
// rows is one contiguous stretch that 1 KiB direct-to-LDS loads fetch; stages stay in flight
// across K steps and tiles.  The epilogue applies the activation in fp32, rounds once, and
// stores 16-byte runs straight from the accumulators (into K-blocked H for GEMM1).
// Few rows per expert, both types (gemm_stream): K cut between a workgroup's waves, weights
// streamed into registers.  Which kernel a call takes: shapes.h.
// fp32, many rows (gemm_f32_lds): 32 x 128 tiles on v_mfma_f32_32x32x2_f32, row-major operands
// in 128-byte row pieces through two direct-to-LDS stages, three workgroups per CU; calls of
// at most 1024 rows split GEMM2's K into parts summed by split_reduce (or, with the combine
// folded in, split_combine) in a fixed order.  gemm_f32 (register-staged 64 x 64 tiles) only
// for an up-projection whose h is not a multiple of 32.
#include "common.h"
#include "kernels.h"
#include "lds_dma.h"
#include "shapes.h"

#include "../../include/moeshard.h"

#include <algorithm>
#include <mutex>
#include <type_traits>

namespace moe {

int device_cus() {
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        return n;
    }();
    return cus;
}

namespace {

enum Epi { kEpiGelu = 0, kEpiGeluTanh = 1, kEpiSwiglu = 2, kEpiNone = 3 };

struct GroupedGemm {
    const void* a;           // [rows][K], or with `gather` [a_rows][K] read through it
    const void* b;           // [E][N rows][K]  (K-contiguous weights)
    const void* b2;          // SwiGLU up projection, same layout as b
    void* c;                 // [rows][ldc]
    const int32_t* offsets;  // [E + 1] row segment of every expert
    int E, K, N, ldc, n_tiles;
    int64_t b_estride;  // elements from one expert's weights to the next
    int64_t rows_max;   // rows of a and c; no row at or past it is touched
    // Up-projection only: grouped row p reads row gather[p] of a (clamped to
    // [0, a_rows)) instead of row p -- the dispatch gather folded into the loads.
    const int32_t* gather;
    int64_t a_rows;
    // Down-projection, top-1 only: grouped row p is stored as w[t] * row into row
    // t = scatter[p] (clamped to [0, c_rows)) of c instead of row p -- Step 5 folded in.
    const int32_t* scatter;
    const float* scatter_w;
    int64_t c_rows;
    // Down-projection only: sums in fp32 to partial[s][row][N] (no scale, no scatter) for a
    // kernel that adds the parts in order.  gemm_f32_lds: with ksplit > 1 every tile as ksplit
    // parts of K / ksplit each.  gemm_stream: whole sums, one part.  The bf16 tiles store theirs
    // as fp32 output (c), so they read neither.
    int ksplit;
    float* partial;
};

// Source row of grouped row p: p itself, or gather[p] clamped into a (entries past the
// assigned rows are never written by the dispatch, so their value is arbitrary).
__device__ __forceinline__ int64_t source_row(const GroupedGemm& g, int64_t p) {
    if (!g.gather) return p;
    const int64_t r = g.gather[p];
    return r < 0 ? 0 : (r >= g.a_rows ? g.a_rows - 1 : r);
}

constexpr int kThreads = 256;

// Exclusive prefix over experts of ceil(count / BM) into tstart[0..E]; returns the total.
// One wave scans (four experts per lane, then a shuffle scan); one barrier publishes it.
template <int BM>
__device__ __forceinline__ int tile_prefix(const int32_t* __restrict__ offsets, int E, int* tstart) {
    static_assert(MOE_MAX_EXPERTS == 4 * 64, "four experts per lane of one wave");
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        // offsets of the lane's four experts and the next, all loaded before any is used
        // (from clamped indices: a load behind a per-lane condition waits for itself)
        int o[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) o[i] = offsets[min(lane * 4 + i, E)];
        int ex[4], run = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int cnt = (lane * 4 + i < E) ? o[i + 1] - o[i] : 0;
            ex[i] = run;
            run += cnt > 0 ? (cnt + BM - 1) / BM : 0;
        }
        int incl = run;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        const int base = incl - run;
#pragma unroll
        for (int i = 0; i < 4; ++i) tstart[lane * 4 + i] = base + ex[i];
        if (lane == 63) tstart[4 * 64] = incl;
    }
    __syncthreads();
    return tstart[E];
}

// Largest expert e with tstart[e] <= mt (an expert that owns row tile mt).
__device__ __forceinline__ int find_expert(const int* tstart, int E, int mt) {
    int lo = 0, hi = E - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tstart[mid] <= mt) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <int EPI>
__device__ __forceinline__ float epilogue(float u, float g) {
    if (EPI == kEpiGelu) return act_gelu(u);
    if (EPI == kEpiGeluTanh) return act_gelu_tanh(u);
    if (EPI == kEpiSwiglu) return silu(u) * g;
    return u;
}

// The same activations for bf16 H (error far below its rounding).  ROWM: up-projections whose h is
// not a multiple of 32 take the forms with no larger an error than erff and expf have (root mean
// square over N(0, 1): GELU 2.1e-8 against 3.9e-8; relative: SiLU 1.4e-7 against 5.5e-7).
template <int EPI, bool ROWM>
__device__ __forceinline__ float epilogue_bf16(float u, float g) {
    if (EPI == kEpiGelu) return ROWM ? act_gelu_near(u) : act_gelu_fast(u);
    if (EPI == kEpiGeluTanh) return act_gelu_tanh_fast(u);
    if (EPI == kEpiSwiglu) return (ROWM ? silu(u) : silu_fast(u)) * g;
    return u;
}

// ------------------------------------------------------------------ bf16 MFMA kernel, direct-to-LDS pipeline
//
// Tile: BM activation rows x BW weight rows (SwiGLU: BW/2 rows of W1 + the same rows of
// W3), K in steps of BK = 32.  A row's 32-element slice is one LDS row of 64 bytes holding
// 4 chunks of 16 bytes; chunk c of row r is stored at position c ^ swz(r), which keeps the
// 32-row MFMA fragment reads free of bank conflicts.  Global data goes straight to LDS with
// global_load_lds_dwordx4 (lane l of a wave instruction fills bytes [16 l, 16 l + 16) of a
// 1 KiB span: 16 LDS rows), NS stages deep.  The weights are K-blocked (see the pack step:
// a stage's rows are one contiguous run), and so is the intermediate H, which the
// up-projection writes and the down-projection reads: every 1 KiB load of those operands
// is 1 KiB of contiguous memory, eight full 128-byte lines.  The up-projection's
// activations (x_perm) are row-major: 64-byte pieces of 16 rows.  The weight fragment is
// the MFMA's first operand, so each lane ends up holding 4 consecutive output columns of
// one row (one 8- or 16-byte store per group).  K must be a multiple of 32.

// WN: waves along the tile's columns (the waves are 2 x WN; 4 or 8 per workgroup).
template <int BM, int BW, int BK, int NS, int EPI, int WN = 2>
struct LdsShape {
    static constexpr bool kDual = (EPI == kEpiSwiglu);
    static constexpr int kNB = kDual ? 2 : 1;
    static constexpr int kBN = BW / kNB;          // output columns per tile
    static constexpr int kWaves = 2 * WN;
    static constexpr int kThreadsWG = 64 * kWaves;
    static constexpr int kMI = BM / 64;           // 32-row blocks per wave (BM / 2 rows)
    static constexpr int kNI = kBN / (32 * WN);   // 32-column blocks per wave per matrix
    static constexpr int kCPR = BK / 8;           // 16-byte chunks per LDS row
    static constexpr int kRPI = 64 / kCPR;        // LDS rows per 1 KiB wave load
    static constexpr int kRows = BM + BW;         // LDS rows per stage
    static constexpr int kLPW = kRows / kRPI / kWaves;  // 1 KiB loads per wave per stage
    static constexpr int kKS = BK / 16;           // MFMA K steps per stage
    static constexpr int kSwzShift = (kCPR == 8) ? 1 : 2;  // rows sharing a 256-byte bank line
    static constexpr size_t kBytes = (size_t)NS * kRows * BK * 2;
    static constexpr int kPerCU = (kBytes <= 80 * 1024) ? 2 : 1;  // workgroups per CU
    static_assert(kMI >= 1 && kNI >= 1 && kBN % (32 * WN) == 0, "tile too small for the waves' 32 x 32 blocks");
    static_assert(kRows % (kRPI * kWaves) == 0, "stage rows must split evenly over the waves");
    static_assert(BM % (kWaves * kRPI) == 0 && kBN % (kWaves * kRPI) == 0, "a wave load carries one kind of row");
    static_assert(BK == 32, "the K-blocked operands come in blocks of 32");
};

// Stores of a 32 x 32 output block.  The MFMA layout leaves lane (row l % 32, half l / 32)
// with columns 8 q + 4 half .. 8 q + 4 half + 3 of its row, q = 0..3.  Stored like that, an
// instruction writes 32 rows in pieces of 32 bytes; the lanes first trade their runs so that
// every instruction writes 64 contiguous bytes of 16 rows: lane l stores rows l % 16 and
// 16 + l % 16 of the block, the same columns of both.  Every lane of the wave must call (the
// lane swaps).  Measured: 1024-column fp32 outputs 32.2 -> 31.2 us (8192 rows, K = 512),
// 4096-column bf16 ones 109.4 -> 106.6 us (8192 rows, K = 1792).
//
// swap(vdst, src) of permlane32: lanes 32..63 of vdst <-> lanes 0..31 of src; of permlane16:
// odd rows of 16 lanes of vdst <-> even rows of src; both return {vdst, src}.
//
// bf16: pk[q] holds the lane's four columns of run q.  After the permlane32 swaps lane l holds
// columns 8 half .. + 7 and 16 + 8 half .. + 7 of its row, after the permlane16 swaps columns
// c .. c + 7, c = store_col_bf16(), of the two rows.  d0 / d1: the rows' addresses there.
__device__ __forceinline__ int store_col_bf16(int lane) { return 8 * (lane >> 5) + 16 * ((lane >> 4) & 1); }
__device__ __forceinline__ void store_block_bf16(bf16_t* d0, bf16_t* d1, const uint2 (&pk)[4], bool ok0, bool ok1) {
    const auto a0 = __builtin_amdgcn_permlane32_swap(pk[0].x, pk[1].x, false, false);
    const auto a1 = __builtin_amdgcn_permlane32_swap(pk[0].y, pk[1].y, false, false);
    const auto b0 = __builtin_amdgcn_permlane32_swap(pk[2].x, pk[3].x, false, false);
    const auto b1 = __builtin_amdgcn_permlane32_swap(pk[2].y, pk[3].y, false, false);
    const auto x = __builtin_amdgcn_permlane16_swap(a0[0], b0[0], false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(a1[0], b1[0], false, false);
    const auto z = __builtin_amdgcn_permlane16_swap(a0[1], b0[1], false, false);
    const auto w = __builtin_amdgcn_permlane16_swap(a1[1], b1[1], false, false);
    if (ok0) *reinterpret_cast<uint4*>(d0) = make_uint4(x[0], y[0], z[0], w[0]);
    if (ok1) *reinterpret_cast<uint4*>(d1) = make_uint4(x[1], y[1], z[1], w[1]);
}

// fp32, runs q = 2 p and 2 p + 1 (u and v): after the swaps the lane holds columns
// 16 p + store_col_f32() .. + 3 of the two rows.
__device__ __forceinline__ int store_col_f32(int lane) { return 4 * (lane >> 5) + 8 * ((lane >> 4) & 1); }
__device__ __forceinline__ void store_block_f32(float* d0, float* d1, const float (&u)[4], const float (&v)[4], bool ok0,
                                                bool ok1) {
    float4 r0, r1;
    float* const o0 = &r0.x;
    float* const o1 = &r1.x;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(u[c]), __float_as_uint(v[c]), false, false);
        o0[c] = __uint_as_float(x[0]);
        o1[c] = __uint_as_float(x[1]);
    }
    if (ok0) *reinterpret_cast<float4*>(d0) = r0;
    if (ok1) *reinterpret_cast<float4*>(d1) = r1;
}

// One accumulator value for the epilogue.  With 256 accumulator registers per lane they
// live in AGPRs, and VALU work needs them in VGPRs; left to itself the compiler copies all of
// them at once when the K loop ends, which needs every VGPR and spills the loop's live
// values.  Reading them one at a time keeps the epilogue's VGPR use small.
template <bool IN_AGPR>
__device__ __forceinline__ float acc_read(float a) {
    if (!IN_AGPR) return a;
    float v;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
    return v;
}

// The row-tile table (first row tile of every expert): in LDS, written by tile_prefix ...
struct LdsTiles {
    const int* tstart;
    int E;
    __device__ __forceinline__ int find(int mt) const { return find_expert(tstart, E, mt); }
    __device__ __forceinline__ int start(int e) const { return tstart[e]; }
};

// ... or in registers, one copy per wave (for kernels whose LDS is all stage buffers): lane l
// holds the first row tile of experts 4 l .. 4 l + 3.  Every lane of the wave must call.
template <int BM>
struct RegTiles {
    int ex[4];
    int E, total;
    __device__ __forceinline__ void build(const int32_t* __restrict__ offsets, int num_experts) {
        static_assert(MOE_MAX_EXPERTS == 4 * 64, "four experts per lane of one wave");
        E = num_experts;
        const int lane = threadIdx.x & 63;
        int o[5];  // loaded together from clamped indices, as in tile_prefix
#pragma unroll
        for (int i = 0; i < 5; ++i) o[i] = offsets[min(lane * 4 + i, num_experts)];
        int run = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int cnt = (lane * 4 + i < E) ? o[i + 1] - o[i] : 0;
            ex[i] = run;
            run += cnt > 0 ? (cnt + BM - 1) / BM : 0;
        }
        int incl = run;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) ex[i] += incl - run;
        total = __builtin_amdgcn_readfirstlane(__shfl(incl, 63, 64));
    }
    // largest expert whose first row tile is <= mt (the table is non-decreasing): a count
    // over the wave by ballots, no cross-lane data movement
    __device__ __forceinline__ int find(int mt) const {
        const int lane = threadIdx.x & 63;
        int c = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) c += __popcll(__ballot(lane * 4 + i < E && ex[i] <= mt));
        return c - 1;
    }
    // e is wave-uniform: read it from lane e / 4
    __device__ __forceinline__ int start(int e) const {
        const int q = e & 3;
        const int v = q == 0 ? ex[0] : q == 1 ? ex[1] : q == 2 ? ex[2] : ex[3];
        return __builtin_amdgcn_readlane(v, e >> 2);
    }
};

// Where a tile's rows are read from.  The tile reads BM activation rows starting at
// row_base and BN weight rows starting at n_base, both shifted back from the tile's own
// first row / column when the tile would run past the end of the buffer (so every load
// stays inside it without a per-row check); the epilogue stores only the tile's own rows
// [row0, row_end) and columns [n0, N).
//
// The load cursor keeps its tile's geometry in scalar registers through the K loop, so it is
// four 32-bit values (a row of H takes at least 256 bytes, so a call that fits the memory has
// fewer than 2^30 rows) and the two bases are derived from them.  With 64-bit rows and stored
// bases gemm_up_pairs<GELU> spilled 30 scalar registers, 15 like this, and the small tiles some;
// 32768 tokens (x 1024 -> 4096 -> 1024) 1263.8 -> 1256.1 us.
struct TileGeom {
    int row0, row_end, n0, e;
};

template <int BM>
__device__ __forceinline__ int row_base(const GroupedGemm& g, const TileGeom& t) {
    return min(max(t.row0, 0), max(static_cast<int>(g.rows_max) - BM, 0));
}
template <int BN>
__device__ __forceinline__ int n_base(const GroupedGemm& g, const TileGeom& t) {
    return min(t.n0, max(g.N - BN, 0));
}

template <int BM, int BN, typename Tiles>
__device__ __forceinline__ TileGeom tile_geom(const GroupedGemm& g, const Tiles& tiles, int L) {
    TileGeom t;
    t.e = __builtin_amdgcn_readfirstlane(tiles.find(L / g.n_tiles));
    const int first = __builtin_amdgcn_readfirstlane(tiles.start(t.e));
    const int seg0 = g.offsets[t.e], seg1 = g.offsets[t.e + 1];
    // tile L of the list is tile l of its expert's m x n_tiles tiles: groups of at most 8 row
    // tiles, as even as they go, column-major inside a group
    const int m = (seg1 - seg0 + BM - 1) / BM;
    const int l = L - first * g.n_tiles;
    const int gsz = (m + (m + 7) / 8 - 1) / ((m + 7) / 8);
    const int grp = l / (gsz * g.n_tiles);
    const int rem = l - grp * gsz * g.n_tiles;
    const int sz = min(gsz, m - grp * gsz);
    const int nt = rem / sz, mt = grp * gsz + rem - nt * sz;
    t.row0 = seg0 + mt * BM;
    t.row_end = min(seg1, static_cast<int>(g.rows_max));
    t.n0 = nt * BN;
    return t;
}

// Last activation row of a tile worth loading: rows past the tile's valid ones then load that
// row again (their results are never stored), so that a mostly empty tile's loads touch one
// line each.  A tile shifted back at the end of the buffer keeps the buffer's limit.
template <int BM>
__device__ __forceinline__ int tile_row_limit(const GroupedGemm& g, const TileGeom& t) {
    const int lim = static_cast<int>(g.rows_max < BM ? g.rows_max : BM) - 1;
    const int valid = t.row_end - t.row0;
    return row_base<BM>(g, t) == t.row0 && valid >= 1 ? min(valid - 1, lim) : lim;
}

// Epilogue of one row of 32 x 32 blocks: rows [row, row + 32) of the wave (row: buffer row of
// the block's first), NI blocks of columns from n_lo, accumulators acc[nb][j].  kUp: bf16 H,
// K-blocked; otherwise row-major C (bf16 or fp32), with `scatter` w[t] * row into row
// t = scatter[row].  Rows outside the tile's and columns outside [t.n0, N) are not stored.
template <int EPI, bool OB, int NB, int NI, bool IN_AGPR, bool ROWM = false, typename Acc>
__device__ __forceinline__ void store_row_block(const GroupedGemm& g, const TileGeom& t, int row, int n_lo,
                                                const Acc& acc) {
    constexpr bool kUp = EPI != kEpiNone;
    const int lane = threadIdx.x & 63;
    const int row_lo = max(t.row0, 0);
    int64_t r0 = row + (lane & 15), r1 = r0 + 16;  // the rows this lane stores
    const bool ok0 = r0 >= row_lo && r0 < t.row_end, ok1 = r1 >= row_lo && r1 < t.row_end;
    float scale = 1.f;
    if (!kUp && g.scatter) {
        // the grouped row's token and gate weight: looked up for the row whose sums this lane
        // holds (row + l % 32), then handed to the lanes that store it
        const int rs = row + (lane & 31);
        const bool ok = rs >= row_lo && rs < t.row_end;
        const int64_t src = ok ? g.scatter[rs] : 0;
        const int tok = static_cast<int>(src < 0 ? 0 : (src >= g.c_rows ? g.c_rows - 1 : src));
        scale = ok ? g.scatter_w[tok] : 0.f;
        r0 = __shfl(tok, lane & 15, 64);
        r1 = __shfl(tok, 16 + (lane & 15), 64);
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int cb = n_lo + j * 32;  // the block's first column
        if (OB) {
            uint2 pk[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    v[c] = epilogue_bf16<EPI, ROWM>(acc_read<IN_AGPR>(acc[0][j][4 * q + c]),
                                                    acc_read<IN_AGPR>(acc[NB - 1][j][4 * q + c]));
                if (!kUp)
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] *= scale;
                pk[q].x = pack_bf16x2(v[0], v[1]);
                pk[q].y = pack_bf16x2(v[2], v[3]);
            }
            // runs of 8 columns: inside one 32-column block of K-blocked H (N, n0 and cb are
            // multiples of 32 there) or inside a row of y (N, n0 and cb are multiples of 8),
            // wholly before n0 or wholly after it
            const int col = cb + store_col_bf16(lane);
            const bool okc = col >= t.n0 && col < g.N;
            bf16_t* const C = static_cast<bf16_t*>(g.c);
            const int64_t hb = (static_cast<int64_t>(cb) >> 5) * g.rows_max;
            bf16_t* const d0 = C + (kUp ? (hb + r0) * 32 + (col & 31) : r0 * g.ldc + col);
            bf16_t* const d1 = C + (kUp ? (hb + r1) * 32 + (col & 31) : r1 * g.ldc + col);
            store_block_bf16(d0, d1, pk, ok0 && okc, ok1 && okc);
        } else {
            // fp32: groups of 4 columns, N % 4 == 0
            float* const C = static_cast<float*>(g.c);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                float u[4], v[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    u[c] = scale * acc_read<IN_AGPR>(acc[0][j][8 * p + c]);
                    v[c] = scale * acc_read<IN_AGPR>(acc[0][j][8 * p + 4 + c]);
                }
                const int col = cb + 16 * p + store_col_f32(lane);
                const bool okc = col >= t.n0 && col < g.N;
                store_block_f32(C + r0 * g.ldc + col, C + r1 * g.ldc + col, u, v, ok0 && okc, ok1 && okc);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // one block at a time: keeps the scheduler from pulling every accumulator into VGPRs
        // at once
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Persistent grouped GEMM.  The grid is a fixed number of workgroups (one or two per CU);
// the tiles are dealt to the 8 XCDs in contiguous runs (the hardware deals workgroups
// round-robin, so workgroup b sits on XCD b % 8) and, inside a run, round-robin to that
// XCD's workgroups, so concurrently running tiles share rows or weights in its L2.
//
// Pipeline (per wave; stage b = the b-th K step this workgroup multiplies, counted across
// tiles).  Loads run NS - 1 stages ahead, across tile boundaries.  Stage b is published by
// one barrier: before it each wave waits for its own loads of stage b (vmcnt) and for its
// own LDS reads of stage b - 1 (lgkmcnt); after it, stage b is complete for every wave and
// nobody reads stage b - 1 any more, so its buffer is refilled with stage b + NS - 1 right
// away.  Inside a tile, that barrier sits in front of the last MFMA step of stage b - 1:
// the first fragments of stage b are read from LDS while those MFMAs run, and every other
// MFMA step's fragments are read during the step before it (two fragment sets in
// registers).  Every 1 KiB load has a fixed per-lane offset (computed once) from a scalar
// base that moves by 2*BK bytes per stage.
//
// The activation epilogues belong to the up-projection (A = x_perm row-major, C = H
// K-blocked); the plain one to the down-projection (A = H K-blocked, C = y_perm row-major).
// RM: weights row-major (h not a multiple of 32): like the activations they come in 64-byte
// pieces of a row, and the last stage's 16-byte chunks past the end of K, of both operands,
// come from sixteen zero bytes instead.
__device__ const uint4 kZeroChunk = {0, 0, 0, 0};

template <int BM, int BW, int BK, int NS, int EPI, bool OB, int WN = 2, bool RM = false>
__global__ __launch_bounds__((LdsShape<BM, BW, BK, NS, EPI, WN>::kThreadsWG),
                             (LdsShape<BM, BW, BK, NS, EPI, WN>::kPerCU))
void gemm_bf16_lds(GroupedGemm g) {
    typedef LdsShape<BM, BW, BK, NS, EPI, WN> S;
    constexpr bool kUp = EPI != kEpiNone;
    constexpr int NB = S::kNB, BN = S::kBN, MI = S::kMI, NI = S::kNI, ROWS = S::kRows, LPW = S::kLPW;
    constexpr int CPR = S::kCPR, RPI = S::kRPI, SH = S::kSwzShift, KS = S::kKS, NW = S::kWaves;
    constexpr int kStageBytes = ROWS * BK * 2;
    constexpr int kAJ = BM / (NW * RPI);  // loads per wave per stage that carry activation rows
    __shared__ int tstart[kThreads + 1];
    extern __shared__ __align__(1024) unsigned char smem_raw[];

    const int total_m = tile_prefix<BM>(g.offsets, g.E, tstart);
    const LdsTiles tiles{tstart, g.E};
    const int total = total_m * g.n_tiles;
    const int per = (total + 7) >> 3;
    const int xcd = blockIdx.x & 7, nslot = gridDim.x >> 3;
    const int t_end = min(total, (xcd + 1) * per);
    const int t_first = xcd * per + static_cast<int>(blockIdx.x >> 3);
    if (t_first >= t_end) return;
    static_assert(!RM || kUp, "H is K-blocked");
    const int nk = RM ? (g.K + BK - 1) / BK : g.K / BK;

    const int tid = threadIdx.x, lane = tid & 63;
    // the wave index is uniform across a wave; say so, so that per-wave choices stay scalar
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)smem_raw)));

    // Per-lane byte offsets of this wave's loads: load j fills LDS rows (NW j + wave) * RPI
    // + lane / CPR of a stage, slot lane % CPR, with global chunk slot ^ swz(row).  Rows past
    // a buffer smaller than one tile repeat its last row.  The weights' are the same for every
    // tile, the activations' (j < kAJ) are set with it.
    uint32_t voff[LPW];
    {
        const int r_lane = lane / CPR, c_lane = lane % CPR;
        const int b_lim = (g.N < BN ? g.N : BN) - 1;
#pragma unroll
        for (int j = kAJ; j < LPW; ++j) {
            const int R = (j * NW + wave) * RPI + r_lane;
            const int kc = c_lane ^ ((R >> SH) & (CPR - 1));
            const uint32_t row_bytes = RM ? static_cast<uint32_t>(2 * g.K) : 64u;
            voff[j] = static_cast<uint32_t>(min((R - BM) % BN, b_lim)) * row_bytes + static_cast<uint32_t>(kc * 16);
        }
    }

    // ---- load cursor: tile lt, K step lk, scalar bases of the tile's rows at K = 0
    int lt = t_first, lk = 0;
    const unsigned char *src_a = nullptr, *src_b0 = nullptr, *src_b1 = nullptr;
    TileGeom lg;  // of the tile being loaded
    auto set_tile = [&](int L) {
        lg = tile_geom<BM, BN>(g, tiles, L);
        const TileGeom& t = lg;
        const int64_t rb = kUp ? 2 * static_cast<int64_t>(g.K) : 64;
        if (kUp && g.gather) {
            // this lane's activation rows come from the gathered source rows (the index
            // load makes the compiler wait for the loads in flight: once per tile)
            const int r_lane = lane / CPR, c_lane = lane % CPR;
            const int a_lim = tile_row_limit<BM>(g, t);
#pragma unroll
            for (int j = 0; j < kAJ; ++j) {
                const int R = (j * NW + wave) * RPI + r_lane;
                const int kc = c_lane ^ ((R >> SH) & (CPR - 1));
                const int64_t src = source_row(g, row_base<BM>(g, t) + min(R, a_lim));
                voff[j] = static_cast<uint32_t>(src) * static_cast<uint32_t>(2 * g.K) + static_cast<uint32_t>(kc * 16);
            }
            src_a = uniform_ptr(g.a);
        } else {
            const int r_lane = lane / CPR, c_lane = lane % CPR;
            const int a_lim = tile_row_limit<BM>(g, t);
#pragma unroll
            for (int j = 0; j < kAJ; ++j) {
                const int R = (j * NW + wave) * RPI + r_lane;
                const int kc = c_lane ^ ((R >> SH) & (CPR - 1));
                voff[j] = static_cast<uint32_t>(min(R, a_lim)) * static_cast<uint32_t>(rb) + static_cast<uint32_t>(kc * 16);
            }
            src_a = uniform_ptr(static_cast<const unsigned char*>(g.a) + row_base<BM>(g, t) * rb);
        }
        const int64_t boff = (t.e * g.b_estride) * 2 + static_cast<int64_t>(n_base<BN>(g, t)) * (RM ? 2 * g.K : 64);
        src_b0 = uniform_ptr(static_cast<const unsigned char*>(g.b) + boff);
        src_b1 = NB > 1 ? uniform_ptr(static_cast<const unsigned char*>(g.b2) + boff) : src_b0;
    };
    int issued = 0;  // stages issued by this wave so far
    auto issue_next = [&]() {
        if (lt >= t_end) return;
        const uint32_t dst = lds0 + (issued % NS) * kStageBytes;
        // K block lk of each operand: the next 64 bytes of every row (row-major x_perm), or
        // the next block of all rows (K-blocked)
        const int64_t ka = kUp ? static_cast<int64_t>(lk) * 64 : static_cast<int64_t>(lk) * g.rows_max * 64;
        const int64_t kb = static_cast<int64_t>(lk) * (RM ? 64 : static_cast<int64_t>(g.N) * 64);
        // a lane's chunk of its row is the same in every load (rows differ by multiples of 16)
        const int kc = (lane % CPR) ^ ((lane / CPR >> SH) & (CPR - 1));
        const bool past = RM && lk * 64 + kc * 16 >= 2 * g.K;
#pragma unroll
        for (int j = 0; j < LPW; ++j) {
            const unsigned char* base = j < kAJ ? src_a + ka : ((NB > 1 && (j - kAJ) * NW * RPI >= BN) ? src_b1 : src_b0) + kb;
            if (RM && lk == nk - 1)
                load_lds16_at(past ? reinterpret_cast<const unsigned char*>(&kZeroChunk) : base + voff[j],
                              dst + (j * NW + wave) * RPI * CPR * 16);
            else
                load_lds16(base, voff[j], dst + (j * NW + wave) * RPI * CPR * 16);
        }
        ++issued;
        if (++lk == nk) {
            lk = 0;
            lt += nslot;
            if (lt < t_end) set_tile(lt);
        }
    };
    set_tile(lt);
#pragma unroll
    for (int st = 0; st < NS - 1; ++st) issue_next();

    // ---- fragments: A block i = activation rows wm*BM/2 + 32 i + l32, B block (nb, j) =
    // weight rows BM + nb*BN + wn*BN/2 + 32 j + l32; K chunk 2 ks + lhi of the stage.  Only
    // the first NV row blocks of the wave are read (the rest hold no valid row).
    const int wm = wave / WN, wn = wave % WN;
    const int l32 = lane & 31, lhi = lane >> 5;
    typedef bf16x8_t Frags[MI + NB * NI];
    auto read_frags = [&](auto nv_tag, int stage_slot, int ks, Frags& f) {
        constexpr int NV = decltype(nv_tag)::value;
        const unsigned char* st = smem_raw + stage_slot * kStageBytes;
        const int ch = 2 * ks + lhi;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int R = wm * (BM / 2) + i * 32 + l32;
            f[i] = *reinterpret_cast<const bf16x8_t*>(st + R * (2 * BK) + ((ch ^ ((R >> SH) & (CPR - 1))) << 4));
        }
        if (NV == 0) return;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int R = BM + nb * BN + wn * (BN / WN) + j * 32 + l32;
                f[MI + nb * NI + j] =
                    *reinterpret_cast<const bf16x8_t*>(st + R * (2 * BK) + ((ch ^ ((R >> SH) & (CPR - 1))) << 4));
            }
    };

    // one workgroup per CU: the accumulators fill the AGPRs (see acc_read)
    constexpr bool kAccInAgpr = S::kPerCU == 1;
    int consumed = 0;
    for (int ct = t_first; ct < t_end; ct += nslot) {
        // the loads are NS - 1 stages ahead: still in this tile unless its K is that short
        const TileGeom t = nk >= NS ? lg : tile_geom<BM, BN>(g, tiles, ct);
        // Row blocks of this wave that hold valid rows.  Valid rows start at the tile's first
        // row unless the tile was shifted back at the end of the buffer; then all count.  The
        // count is rounded up to MI / 2 or MI so that three loop bodies cover every case.
        int nv = MI;
        if (row_base<BM>(g, t) == t.row0) {
            const int left = t.row_end - (t.row0 + wm * (BM / 2));
            nv = left <= 0 ? 0 : (left > (MI / 2) * 32 ? MI : MI / 2);
        }
        nv = __builtin_amdgcn_readfirstlane(nv);

        f32x16_t acc[MI][NB][NI];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][nb][j][r] = 0.f;

        // publish the tile's first stage; after an epilogue its stores share the counter
        if (ct != t_first) wait_vmcnt<0>();
        else wait_stages<LPW, NS>(issued - consumed - 1);
        stage_barrier();
        issue_next();

        // the K loop with the MFMAs of the first NV row blocks; every wave takes part in the
        // loads, waits and barriers whatever its NV
        auto k_loop = [&](auto nv_tag) {
            constexpr int NV = decltype(nv_tag)::value;
            // weight block outer, row block inner: consecutive MFMAs share their first operand
            auto mma = [&](const Frags& f) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int j = 0; j < NI; ++j)
#pragma unroll
                        for (int i = 0; i < NV; ++i)
                            acc[i][nb][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[MI + nb * NI + j], f[i],
                                                                                    acc[i][nb][j], 0, 0, 0);
            };
            Frags f0, f1;
            read_frags(nv_tag, consumed % NS, 0, f0);
            for (int ck = 0; ck < nk; ++ck) {
                const int slot = consumed % NS;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    Frags& cur = (ks & 1) ? f1 : f0;
                    Frags& nxt = (ks & 1) ? f0 : f1;
                    if (ks + 1 < KS) {
                        read_frags(nv_tag, slot, ks + 1, nxt);
                    } else if (ck + 1 < nk) {
                        // publish stage consumed + 1 (see above), refill, start its fragments
                        wait_lgkm0();
                        wait_stages<LPW, NS>(issued - consumed - 2);
                        stage_barrier();
                        issue_next();
                        read_frags(nv_tag, (consumed + 1) % NS, 0, nxt);
                    }
                    if (NV > 0) {
                        mma(cur);
                        interleave_reads<NB * NV * NI, NV + NB * NI>();
                    }
                }
                // KS is even for BK 32 / 64, so the next step's first fragments are in f0
                ++consumed;
            }
        };
        if (nv == MI) k_loop(std::integral_constant<int, MI>());
        else if (nv > 0) k_loop(std::integral_constant<int, MI / 2>());
        else k_loop(std::integral_constant<int, 0>());

        // ---- epilogue of tile ct
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if (i >= nv) break;  // no valid row in this block or any later one
            store_row_block<EPI, OB, NB, NI, kAccInAgpr, RM>(g, t, row_base<BM>(g, t) + wm * (BM / 2) + i * 32,
                                                             n_base<BN>(g, t) + wn * (BN / WN), acc[i]);
        }
    }
}
// ------------------------------------------------------------------ bf16 up-projection, paired A stages
//
// The up-projection's activations are rows of x (gathered through row_src) or of x_perm,
// row-major, so the kernel above reads them as 64-byte pieces: half a 128-byte line per
// stage, the other half a stage later.  This variant (K % 64 == 0) loads 128 bytes of an
// activation row for two stages at once.  The A side has two 16 KiB slots of 128 rows x
// 128 bytes (one in use, one filling; chunk c of row r sits at c ^ (r % 8), so the 8 rows
// that 8 lanes of a fragment read touch fall on 8 different bank groups); the weights keep
// the three-stage ring of K-blocked 256-row stages.  That is 80 KiB, two workgroups per CU
// with nothing left over, so the row-tile table is kept in registers.  Even stages issue 4
// A and 4 B loads per wave, odd stages 4 B loads; the vmcnt waits count them that way.
// Fragments, MFMA order and epilogue are those of gemm_bf16_lds<128, 256, 32, 3, EPI,
// true>, and so is every output bit.
constexpr int kUpASlot = 128 * 128;                       // bytes of one A slot
constexpr int kUpBSlot = 256 * 64;                        // bytes of one B stage
constexpr size_t kUpPairBytes = 2 * kUpASlot + 3 * kUpBSlot;  // 80 KiB

template <int EPI>
__global__ __launch_bounds__(kThreads, 2) void gemm_up_pairs(GroupedGemm g) {
    constexpr int BM = 128, BW = 256, NS = 3;
    typedef LdsShape<BM, BW, 32, NS, EPI> S;
    constexpr int NB = S::kNB, BN = S::kBN, MI = S::kMI, NI = S::kNI, KS = S::kKS;
    constexpr int kBBase = 2 * kUpASlot;
    constexpr int LPA = BM / 8 / 4;   // 1 KiB loads per wave of an A pair (8 rows x 128 bytes)
    constexpr int LPB = BW / 16 / 4;  // 1 KiB loads per wave of a B stage (16 rows x 64 bytes)
    static_assert(kUpPairBytes <= 80 * 1024, "two workgroups per CU");
    extern __shared__ __align__(1024) unsigned char smem_raw[];

    RegTiles<BM> tiles;
    tiles.build(g.offsets, g.E);
    const int total_m = tiles.total;
    const int total = total_m * g.n_tiles;
    const int per = (total + 7) >> 3;
    const int xcd = blockIdx.x & 7, nslot = gridDim.x >> 3;
    const int t_end = min(total, (xcd + 1) * per);
    const int t_first = xcd * per + static_cast<int>(blockIdx.x >> 3);
    if (t_first >= t_end) return;
    const int nk = g.K / 32;  // even: the host runs this kernel only for K % 64 == 0

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds0 = lds_address(smem_raw);
    const int b_lim = (g.N < BN ? g.N : BN) - 1;

    // B: load j fills B rows (4 j + wave) 16 + lane / 4 of a stage, slot lane % 4, with global
    // chunk slot ^ ((row / 4) % 4); the same for every tile
    uint32_t voffB[LPB];
#pragma unroll
    for (int j = 0; j < LPB; ++j) {
        const int R = (j * 4 + wave) * 16 + (lane >> 2);
        const int kc = (lane & 3) ^ ((R >> 2) & 3);
        voffB[j] = static_cast<uint32_t>(min(R % BN, b_lim)) * 64u + static_cast<uint32_t>(kc * 16);
    }
    // A: load j fills A rows (4 j + wave) 8 + lane / 8 of a slot, slot lane % 8, with global
    // chunk slot ^ (row % 8); set per tile
    uint32_t voffA[LPA];

    int lt = t_first, lk = 0;
    const unsigned char *src_a = nullptr, *src_b0 = nullptr, *src_b1 = nullptr;
    TileGeom lg;  // of the tile being loaded
    auto set_tile = [&](int L) {
        lg = tile_geom<BM, BN>(g, tiles, L);
        const TileGeom& t = lg;
#pragma unroll
        for (int j = 0; j < LPA; ++j) {
            const int R = (j * 4 + wave) * 8 + (lane >> 3);
            const int c = (lane & 7) ^ (R & 7);
            // gathered: absolute source row (T h s < 4 GiB is checked by the host); else the
            // tile's base carries the row offset
            const int a_lim_t = tile_row_limit<BM>(g, t);
            const int64_t r = g.gather ? source_row(g, row_base<BM>(g, t) + min(R, a_lim_t)) : min(R, a_lim_t);
            voffA[j] = static_cast<uint32_t>(r) * static_cast<uint32_t>(2 * g.K) + static_cast<uint32_t>(c * 16);
        }
        src_a = uniform_ptr(static_cast<const unsigned char*>(g.a) + (g.gather ? 0 : static_cast<int64_t>(row_base<BM>(g, t)) * 2 * g.K));
        const int64_t boff = (t.e * g.b_estride) * 2 + static_cast<int64_t>(n_base<BN>(g, t)) * 64;
        src_b0 = uniform_ptr(static_cast<const unsigned char*>(g.b) + boff);
        src_b1 = NB > 1 ? uniform_ptr(static_cast<const unsigned char*>(g.b2) + boff) : src_b0;
    };
    int issued = 0;  // stages issued by this wave so far (even at every tile start: nk is even)
    auto issue_next = [&]() {
        if (lt >= t_end) return;
        if ((lk & 1) == 0) {
            // the next 128 bytes of every activation row: K blocks lk and lk + 1
            const uint32_t da = lds0 + ((issued >> 1) & 1) * kUpASlot;
#pragma unroll
            for (int j = 0; j < LPA; ++j)
                load_lds16(src_a + static_cast<int64_t>(lk) * 64, voffA[j], da + (j * 4 + wave) * 1024);
        }
        const uint32_t db = lds0 + kBBase + (issued % NS) * kUpBSlot;
        const int64_t kb = static_cast<int64_t>(lk) * g.N * 64;
#pragma unroll
        for (int j = 0; j < LPB; ++j)
            load_lds16(((NB > 1 && j * 4 * 16 >= BN) ? src_b1 : src_b0) + kb, voffB[j], db + (j * 4 + wave) * 1024);
        ++issued;
        if (++lk == nk) {
            lk = 0;
            lt += nslot;
            if (lt < t_end) set_tile(lt);
        }
    };
    // wait until stage `st` is in LDS while `newer` later stages stay in flight
    auto wait_stage = [&](int st, int newer) {
        if (newer >= 2) wait_vmcnt<LPA + 2 * LPB>();
        else if (newer == 1 && ((st + 1) & 1) == 0) wait_vmcnt<LPA + LPB>();
        else if (newer == 1) wait_vmcnt<LPB>();
        else wait_vmcnt<0>();
    };
    set_tile(lt);
#pragma unroll
    for (int st = 0; st < NS - 1; ++st) issue_next();

    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lhi = lane >> 5;
    typedef bf16x8_t Frags[MI + NB * NI];
    // fragments of stage st (its A slot and half of the slot's rows, its B ring slot)
    auto read_frags = [&](auto nv_tag, int st, int ks, Frags& f) {
        constexpr int NV = decltype(nv_tag)::value;
        const unsigned char* sa = smem_raw + ((st >> 1) & 1) * kUpASlot;
        const int ca = (st & 1) * 4 + 2 * ks + lhi;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int R = wm * (BM / 2) + i * 32 + l32;
            f[i] = *reinterpret_cast<const bf16x8_t*>(sa + R * 128 + ((ca ^ (R & 7)) << 4));
        }
        if (NV == 0) return;
        const unsigned char* sb = smem_raw + kBBase + (st % NS) * kUpBSlot;
        const int cb = 2 * ks + lhi;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int R = nb * BN + wn * (BN / 2) + j * 32 + l32;
                f[MI + nb * NI + j] = *reinterpret_cast<const bf16x8_t*>(sb + R * 64 + ((cb ^ ((R >> 2) & 3)) << 4));
            }
    };

    int consumed = 0;
    for (int ct = t_first; ct < t_end; ct += nslot) {
        const TileGeom t = nk >= NS ? lg : tile_geom<BM, BN>(g, tiles, ct);  // as in gemm_bf16_lds
        int nv = MI;
        if (row_base<BM>(g, t) == t.row0) {
            const int left = t.row_end - (t.row0 + wm * (BM / 2));
            nv = left <= 0 ? 0 : (left > (MI / 2) * 32 ? MI : MI / 2);
        }
        nv = __builtin_amdgcn_readfirstlane(nv);

        f32x16_t acc[MI][NB][NI];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][nb][j][r] = 0.f;

        // publish the tile's first stage; after an epilogue its stores share the counter
        if (ct != t_first) wait_vmcnt<0>();
        else wait_stage(consumed, issued - consumed - 1);
        stage_barrier();
        issue_next();

        auto k_loop = [&](auto nv_tag) {
            constexpr int NV = decltype(nv_tag)::value;
            auto mma = [&](const Frags& f) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int j = 0; j < NI; ++j)
#pragma unroll
                        for (int i = 0; i < NV; ++i)
                            acc[i][nb][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[MI + nb * NI + j], f[i],
                                                                                    acc[i][nb][j], 0, 0, 0);
            };
            Frags f0, f1;
            read_frags(nv_tag, consumed, 0, f0);
            for (int ck = 0; ck < nk; ++ck) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    Frags& cur = (ks & 1) ? f1 : f0;
                    Frags& nxt = (ks & 1) ? f0 : f1;
                    if (ks + 1 < KS) {
                        read_frags(nv_tag, consumed, ks + 1, nxt);
                    } else if (ck + 1 < nk) {
                        wait_lgkm0();
                        wait_stage(consumed + 1, issued - consumed - 2);
                        stage_barrier();
                        issue_next();
                        read_frags(nv_tag, consumed + 1, 0, nxt);
                    }
                    if (NV > 0) {
                        mma(cur);
                        interleave_reads<NB * NV * NI, NV + NB * NI>();
                    }
                }
                ++consumed;
            }
        };
        if (nv == MI) k_loop(std::integral_constant<int, MI>());
        else if (nv > 0) k_loop(std::integral_constant<int, MI / 2>());
        else k_loop(std::integral_constant<int, 0>());

        // epilogue: as in gemm_bf16_lds (bf16 H, K-blocked)
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if (i >= nv) break;
            store_row_block<EPI, true, NB, NI, false>(g, t, row_base<BM>(g, t) + wm * (BM / 2) + i * 32,
                                                      n_base<BN>(g, t) + wn * (BN / 2), acc[i]);
        }
    }
}

// ------------------------------------------------------------------ bf16 MFMA kernel, two wave groups in turn
//
// For calls whose experts have many rows (which calls: turns_up, turns_down in shapes.h), where the
// matrix cores are the bound.  256 x 256 tiles (SwiGLU: 128 columns of W1 and the same of W3),
// eight waves in one workgroup per CU: per product two thirds of the LDS fills (and so of the
// L2 reads) of the 128 x 256 tiles above.  K advances 32 at a time through a ring of four
// 32 KiB stages, three in flight.
//
// The waves form two groups of four, one wave of each group per SIMD.  Group r multiplies the
// tile's odd or even 32-row blocks (so that a tile with few rows still feeds both), wave w of
// it columns 64 w .. 64 w + 63.  The groups take turns: while one runs a stage's 16 MFMAs, the
// other reads its fragments of a stage and issues its share of the loads.  Left to themselves
// both waves of a SIMD read at the same time and then multiply at the same time.  Turns are
// separated by barriers of the whole workgroup; group 1 starts one barrier late.  In turns
// t = 0, 1, ..: group 0 reads stage s in turn 2 s and multiplies it in turn 2 s + 1, group 1
// each one turn later.  So stage s has to be in LDS at the end of turn 2 s - 1: there each wave
// waits for its own loads of it (group 0 after its MFMAs, group 1 after its reads).  Stage s's
// buffer has been read by the end of turn 2 s + 1 and is refilled in each group's reading turn
// of stage s + 1.
//
// Measured, 65536 rows in two experts (x 1024 -> 4096 -> 1024, GELU): down-projection 430 us,
// 1.28 PFLOP/s, and 349 us on zeros, so the rest is power; the 128 x 256 tiles take 521 us.
// The up-projection's epilogue (16 k cycles of vector work a tile and SIMD) has nothing to
// overlap with here, so that short K loops stay with gemm_up_pairs.
constexpr int kTurnStages = 4;
constexpr size_t kTurnBytes = static_cast<size_t>(kTurnStages) * 512 * 64;

template <int EPI, bool OB>
__global__ __launch_bounds__(512, 2) void gemm_turns(GroupedGemm g) {
    constexpr bool kUp = EPI != kEpiNone;
    constexpr int BM = 256, BW = 256, NS = kTurnStages;
    constexpr int NB = EPI == kEpiSwiglu ? 2 : 1;
    constexpr int BN = BW / NB;           // output columns per tile
    constexpr int MI = 4, NI = 2 / NB;    // 32-row / 32-column blocks per wave (and matrix)
    constexpr int LPW = 4;                // 1 KiB loads per wave and stage: two of A, two of B
    constexpr int kStageBytes = (BM + BW) * 64;
    extern __shared__ __align__(1024) unsigned char smem_raw[];

    RegTiles<BM> tiles;
    tiles.build(g.offsets, g.E);
    // This XCD's tiles [t_begin, t_end), dealt round-robin to its workgroups.  A last round
    // that leaves most of them idle is cut finer: its `rest` tiles as `parts` items each, by rows.
    const int total = tiles.total * g.n_tiles, per = (total + 7) >> 3;
    const int xcd = blockIdx.x & 7, nslot = gridDim.x >> 3;
    const int t_begin = min(total, xcd * per), t_end = min(total, t_begin + per);
    const int rest = (t_end - t_begin) % nslot;
    const int parts = rest * 4 <= nslot ? 4 : (rest * 2 <= nslot ? 2 : 1);
    const int whole = t_end - t_begin - rest, items = whole + rest * parts;
    const int i_first = static_cast<int>(blockIdx.x >> 3);
    if (i_first >= items) return;
    auto item_geom = [&](int i) {
        if (i < whole) return tile_geom<BM, BN>(g, tiles, t_begin + i);
        const int r = (i - whole) / parts, p = i - whole - r * parts;
        TileGeom t = tile_geom<BM, BN>(g, tiles, t_begin + whole + r);
        if (parts > 1) {
            // rows [p q, (p + 1) q) of the tile's valid ones, q a multiple of 32
            const int valid = min(t.row_end - t.row0, BM);
            const int q = (valid + 32 * parts - 1) / (32 * parts) * 32;
            t.row_end = min(t.row0 + (p + 1) * q, t.row_end);
            t.row0 += p * q;
        }
        return t;
    };
    const int nk = g.K / 32;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds0 = lds_address(smem_raw);
    const int b_lim = (g.N < BN ? g.N : BN) - 1;

    // load j of a stage fills LDS rows (8 j + wave) 16 + lane / 4, slot lane % 4, with global
    // chunk slot ^ ((row / 4) % 4)
    uint32_t voff[LPW];
    const int r_lane = lane >> 2;
    const uint32_t kc16 = static_cast<uint32_t>(((lane & 3) ^ ((r_lane >> 2) & 3)) * 16);
#pragma unroll
    for (int j = 2; j < LPW; ++j) {
        const int R = ((j - 2) * 8 + wave) * 16 + r_lane;
        voff[j] = static_cast<uint32_t>(min(R % BN, b_lim)) * 64u + kc16;
    }

    int li = i_first, lk = 0;
    TileGeom lg;  // of the item being loaded
    const unsigned char *src_a = nullptr, *src_b0 = nullptr, *src_b1 = nullptr;
    auto set_item = [&](int i) {
        lg = item_geom(i);
        const TileGeom& t = lg;
        const int a_lim = tile_row_limit<BM>(g, t);
        const uint32_t rb = kUp ? static_cast<uint32_t>(2 * g.K) : 64u;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int R = min((j * 8 + wave) * 16 + r_lane, a_lim);
            const int64_t r = (kUp && g.gather) ? source_row(g, row_base<BM>(g, t) + R) : R;
            voff[j] = static_cast<uint32_t>(r) * rb + kc16;
        }
        src_a = uniform_ptr(static_cast<const unsigned char*>(g.a) +
                            ((kUp && g.gather) ? 0 : row_base<BM>(g, t) * static_cast<int64_t>(rb)));
        const int64_t boff = (t.e * g.b_estride) * 2 + static_cast<int64_t>(n_base<BN>(g, t)) * 64;
        src_b0 = uniform_ptr(static_cast<const unsigned char*>(g.b) + boff);
        src_b1 = NB > 1 ? uniform_ptr(static_cast<const unsigned char*>(g.b2) + boff) : src_b0;
    };
    int issued = 0, slot_w = 0;  // stages issued so far; their ring slot
    const int64_t a_step = kUp ? 64 : g.rows_max * 64, b_step = static_cast<int64_t>(g.N) * 64;
    auto issue_next = [&]() {
        if (li >= items) return;
        const uint32_t dst = lds0 + slot_w * kStageBytes + wave * 1024;
        load_lds16(src_a, voff[0], dst);
        load_lds16(src_a, voff[1], dst + 8 * 1024);
        load_lds16(src_b0, voff[2], dst + 16 * 1024);
        load_lds16(NB > 1 ? src_b1 : src_b0, voff[3], dst + 24 * 1024);
        src_a += a_step;
        src_b0 += b_step;
        if (NB > 1) src_b1 += b_step;
        ++issued;
        slot_w = slot_w + 1 == NS ? 0 : slot_w + 1;
        if (++lk == nk) {
            lk = 0;
            li += nslot;
            if (li < items) set_item(li);
        }
    };
    set_item(li);
#pragma unroll
    for (int st = 0; st < NS - 1; ++st) issue_next();

    const int grp = wave >> 2, wn = wave & 3;
    const int l32 = lane & 31, lhi = lane >> 5;
    // a fragment's byte offset inside its 32 LDS rows: K chunk 2 ks + lhi of row l32
    const uint32_t f0 = static_cast<uint32_t>(l32 * 64 + ((lhi ^ ((l32 >> 2) & 3)) << 4));
    const uint32_t f1 = static_cast<uint32_t>(l32 * 64 + (((2 + lhi) ^ ((l32 >> 2) & 3)) << 4));

    int consumed = 0, slot_r = 0;
    wait_stages<LPW, NS>(issued - 1);
    stage_barrier();
    if (grp == 1) stage_barrier();
    for (int ci = i_first; ci < items; ci += nslot) {
        // the loads are NS - 1 stages ahead: still in this item unless it is that short
        const TileGeom t = nk >= NS ? lg : item_geom(ci);
        int nv = MI;
        if (row_base<BM>(g, t) == t.row0) {
            const int left = t.row_end - t.row0 - 32 * grp;
            nv = left <= 0 ? 0 : (left >= BM - 64 ? MI : (left + 63) >> 6);
        }
        nv = __builtin_amdgcn_readfirstlane(nv);

        f32x16_t acc[MI][NB][NI];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][nb][j][r] = 0.f;

        auto k_loop = [&](auto nv_tag) {
            constexpr int NV = decltype(nv_tag)::value;
            for (int ck = 0; ck < nk; ++ck) {
                // ---- memory turn
                bf16x8_t fa[2][MI], fb[2][2];
                const unsigned char* sa = smem_raw + slot_r * kStageBytes + grp * 32 * 64;
                const unsigned char* sb = smem_raw + slot_r * kStageBytes + BM * 64 + wn * (64 / NB) * 64;
                if (NV > 0) {
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) {
                        const uint32_t f = ks ? f1 : f0;
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            fb[ks][j] = *reinterpret_cast<const bf16x8_t*>(sb + f + (NB > 1 ? j * BN * 64 : j * 32 * 64));
#pragma unroll
                        for (int i = 0; i < NV; ++i)
                            fa[ks][i] = *reinterpret_cast<const bf16x8_t*>(sa + f + i * 64 * 64);
                    }
                }
                issue_next();
                ++consumed;
                slot_r = slot_r + 1 == NS ? 0 : slot_r + 1;
                wait_lgkm0();
                if (grp == 1) wait_stages<LPW, NS>(issued - consumed - 1);
                __builtin_amdgcn_sched_barrier(0);
                stage_barrier();
                __builtin_amdgcn_sched_barrier(0);
                // ---- matrix turn
                if (NV > 0) {
                    __builtin_amdgcn_s_setprio(1);
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
#pragma unroll
                            for (int i = 0; i < NV; ++i) {
                                f32x16_t& a = acc[i][NB > 1 ? j : 0][NB > 1 ? 0 : j];
                                a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks][j], fa[ks][i], a, 0, 0, 0);
                            }
                    __builtin_amdgcn_s_setprio(0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (grp == 0) wait_stages<LPW, NS>(issued - consumed - 1);
                stage_barrier();
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (nv == MI) k_loop(std::integral_constant<int, MI>());
        else if (nv == 3) k_loop(std::integral_constant<int, 3>());
        else if (nv == 2) k_loop(std::integral_constant<int, 2>());
        else if (nv == 1) k_loop(std::integral_constant<int, 1>());
        else k_loop(std::integral_constant<int, 0>());

#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if (i >= nv) break;
            store_row_block<EPI, OB, NB, NI, false>(g, t, row_base<BM>(g, t) + (2 * i + grp) * 32, n_base<BN>(g, t) + wn * (BN / 4),
                                                    acc[i]);
        }
    }
    if (grp == 0) stage_barrier();
}

// ------------------------------------------------------------------ fp32 kernel
//
// 64 x 64 tiles on the fp32 matrix cores: four waves, each one 32 x 32 block of
// v_mfma_f32_32x32x2_f32 (lane l supplies A[row l % 32][k l / 32] and B[k l / 32][column
// l % 32] of a two-wide K step, and ends holding column l % 32 of the block).  K advances
// 32 at a time through two LDS buffers stored K-major ([k][row], 4 floats of padding),
// each filled from registers loaded two steps earlier (two register sets take turns), so
// a step's MFMAs overlap the loads of the next two.  Gathered rows are looked up once.

constexpr int kFBM = 64, kFBN = 64, kFBK = 32, kFLD = kFBM + 4;

template <int EPI, bool OB>
__global__ __launch_bounds__(kThreads) void gemm_f32(GroupedGemm g) {
    constexpr int NB = (EPI == kEpiSwiglu) ? 2 : 1;
    __shared__ int tstart[kThreads + 1];
    __shared__ __align__(16) float As[2][kFBK][kFLD];
    __shared__ __align__(16) float Bs[2][NB][kFBK][kFLD];

    const int total = tile_prefix<kFBM>(g.offsets, g.E, tstart);
    const int tile = blockIdx.x;
    const int mt = tile / g.n_tiles;
    const int nt = tile - mt * g.n_tiles;
    if (mt >= total) return;
    const int e = find_expert(tstart, g.E, mt);
    const int64_t row0 = g.offsets[e] + static_cast<int64_t>(mt - tstart[e]) * kFBM;
    const int64_t row_end = g.offsets[e + 1] < g.rows_max ? g.offsets[e + 1] : g.rows_max;
    if (row0 < 0 || row0 >= row_end) return;
    const int n0 = nt * kFBN;
    const float* __restrict__ A = static_cast<const float*>(g.a);
    const float* __restrict__ Bm[NB];
    Bm[0] = static_cast<const float*>(g.b) + e * g.b_estride;
    if (NB > 1) Bm[NB - 1] = static_cast<const float*>(g.b2) + e * g.b_estride;

    // loader: thread t brings rows t / 8 and t / 8 + 32, K values 4 (t % 8) .. + 3 of the step
    // (K % 4 == 0, so a float4 never straddles the end of K)
    const int tid = threadIdx.x;
    const int lrow = tid >> 3, lk = (tid & 7) * 4;
    const float* arow[2];  // this thread's two activation rows (null: past the segment)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int64_t ar = row0 + lrow + 32 * h;
        arow[h] = ar < row_end ? A + source_row(g, ar) * g.K : nullptr;
    }
    struct Regs {
        float4 a[2], b[NB][2];
    };
    const int nk = (g.K + kFBK - 1) / kFBK;
    auto gload = [&](Regs& R, int kt) {
        const int k = kt * kFBK + lk;
        const bool kv = k < g.K;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            R.a[h] = (arow[h] && kv) ? *reinterpret_cast<const float4*>(arow[h] + k) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int n = n0 + lrow + 32 * h;
                R.b[nb][h] = (n < g.N && kv)
                                 ? *reinterpret_cast<const float4*>(Bm[nb] + static_cast<int64_t>(n) * g.K + k)
                                 : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
    };
    auto sstore = [&](const Regs& R, int buf) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = lrow + 32 * h;
            As[buf][lk + 0][r] = R.a[h].x;
            As[buf][lk + 1][r] = R.a[h].y;
            As[buf][lk + 2][r] = R.a[h].z;
            As[buf][lk + 3][r] = R.a[h].w;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                Bs[buf][nb][lk + 0][r] = R.b[nb][h].x;
                Bs[buf][nb][lk + 1][r] = R.b[nb][h].y;
                Bs[buf][nb][lk + 2][r] = R.b[nb][h].z;
                Bs[buf][nb][lk + 3][r] = R.b[nb][h].w;
            }
        }
    };

    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lhi = lane >> 5;
    f32x16_t acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nb][r] = 0.f;

    // step kt: MFMAs on LDS buffer kt % 2; register set `next` holds step kt + 1 and goes to
    // the other buffer after them (that buffer was last read before the previous step's
    // barrier), then takes the loads of step kt + 3
    // a wave whose 32 rows all lie past the segment skips its MFMAs (it still loads and
    // takes part in the barriers); its block is never stored
    const bool live = row0 + wm * 32 < row_end;
    auto step = [&](int kt, Regs& next) {
        const int buf = kt & 1;
        if (live) {
#pragma unroll
            for (int ks = 0; ks < kFBK / 2; ++ks) {
                const float a = As[buf][2 * ks + lhi][wm * 32 + l32];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, Bs[buf][nb][2 * ks + lhi][wn * 32 + l32],
                                                                   acc[nb], 0, 0, 0);
            }
        }
        if (kt + 1 < nk) sstore(next, buf ^ 1);
        __syncthreads();
        if (kt + 3 < nk) gload(next, kt + 3);
    };
    Regs r0, r1;
    gload(r0, 0);
    sstore(r0, 0);
    if (nk > 1) gload(r1, 1);
    if (nk > 2) gload(r0, 2);
    __syncthreads();
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        step(kt, r1);      // r1 holds step kt + 1, then loads kt + 3
        step(kt + 1, r0);  // r0 holds step kt + 2, then loads kt + 4
    }
    if (kt < nk) step(kt, r1);

    // epilogue: register r holds row 8 (r / 4) + 4 lhi + r % 4 of the wave's block; for a
    // fixed r the 32 lanes of a half-wave store 32 consecutive columns
    const int n = n0 + wn * 32 + l32;
    if (n >= g.N) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        int64_t row = row0 + wm * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
        if (row >= row_end) continue;
        float scale = 1.f;
        if (g.scatter) {
            const int64_t src = g.scatter[row];
            row = src < 0 ? 0 : (src >= g.c_rows ? g.c_rows - 1 : src);
            scale = g.scatter_w[row];
        }
        const float v = scale * epilogue<EPI>(acc[0][r], acc[NB - 1][r]);
        if (OB) static_cast<bf16_t*>(g.c)[row * g.ldc + n] = f32_to_bf16(v);
        else static_cast<float*>(g.c)[row * g.ldc + n] = v;
    }
}

// ------------------------------------------------------------------ fp32 pipelined kernel
//
// fp32 operands whose K is a multiple of 32 (every down-projection; the up-projection when
// h % 32 == 0).  Tiles of 32 activation rows x 128 weight rows of each matrix; four waves,
// wave w owning output columns 32 w .. 32 w + 31 of the tile in every matrix.
// v_mfma_f32_32x32x2_f32 takes the weights as its first operand, so a lane ends up holding
// one activation row and, in each group of four registers, four consecutive output columns.
// K advances 32 values (128 bytes of every row) per stage; a stage goes straight to LDS as
// 1 KiB direct loads of 8 rows x 128 bytes, NS stages with NS - 1 in flight across K steps
// and work items (the bf16 kernel's pipeline).  Inside a stage a lane reads, for each group
// of 8 K values, 4 consecutive K values of its row as one 16-byte fragment and feeds element
// c to the c-th of four MFMAs; the other half-wave supplies the group's other 4 K values, so
// the four MFMAs together sum over the whole group.  32-row tiles hold at least one valid
// row each, and an expert's rows waste at most 31 padded rows.  Persistent grid: work items
// (tile, K part) are dealt to the XCDs in contiguous runs and round-robin to each XCD's
// workgroups.  Two stages (one in flight): with one matrix a workgroup needs 40 KiB and
// three share a CU (three waves per SIMD hide each other's waits; measured 3 % faster on a
// 512-token top-1 step than three stages at two per CU), with two matrices 72 KiB and two.
constexpr int kF2BM = 32, kF2BN = 128, kF2BK = 32;  // kF2BK counts floats: 128-byte row pieces

template <int NB>
struct F32Shape {
    static constexpr int kRows = kF2BM + NB * kF2BN;  // LDS rows per stage
    static constexpr int kStageBytes = kRows * kF2BK * 4;
    static constexpr int kLPW = kRows / 8 / 4;         // 1 KiB loads per wave per stage
    static constexpr int kStages = 2;
    static constexpr size_t kBytes = static_cast<size_t>(kStages) * kStageBytes;
    static constexpr int kPerCU = NB == 1 ? 3 : 2;      // workgroups per CU (160 KiB of LDS)
    static_assert(kPerCU * kBytes <= 160 * 1024, "LDS per CU");
};

template <int EPI, bool OB>
__global__ __launch_bounds__(kThreads, (F32Shape<(EPI == kEpiSwiglu) ? 2 : 1>::kPerCU)) void gemm_f32_lds(GroupedGemm g) {
    constexpr int NB = (EPI == kEpiSwiglu) ? 2 : 1;
    typedef F32Shape<NB> S;
    constexpr int BM = kF2BM, BN = kF2BN, LPW = S::kLPW, NS = S::kStages;
    constexpr int kStageBytes = S::kStageBytes;
    constexpr bool kUp = EPI != kEpiNone;
    static_assert(LPW == 1 + 4 * NB, "load 0 carries the 32 activation rows, loads 4 nb + 1 .. 4 nb + 4 matrix nb");
    __shared__ int tstart[kThreads + 1];
    extern __shared__ __align__(1024) unsigned char smem_raw[];

    const int total_m = tile_prefix<BM>(g.offsets, g.E, tstart);
    const LdsTiles tiles{tstart, g.E};
    // work item L: tile L / ks, K part L % ks (ks = 1 unless the down-projection is split)
    const int ks = (!kUp && g.ksplit > 1) ? g.ksplit : 1;
    const int total = total_m * g.n_tiles * ks;
    const int per = (total + 7) >> 3;
    const int xcd = blockIdx.x & 7, nslot = gridDim.x >> 3;
    const int t_first = xcd * per + static_cast<int>(blockIdx.x >> 3);
    const int t_end = min(total, xcd * per + per);
    if (t_first >= t_end) return;
    const int nk = g.K / kF2BK / ks;  // stages per work item

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds0 = lds_address(smem_raw);

    // Per-lane byte offsets of this wave's loads: load j fills LDS rows 8 (4 j + wave) + lane
    // / 8 of a stage, 16-byte slot lane % 8, from global slot (lane % 8) ^ swz(row).  Rows past
    // a buffer smaller than one tile repeat its last row.
    const int r_lane = lane >> 3;
    const int a_lim = static_cast<int>(g.rows_max < BM ? g.rows_max : BM) - 1;
    const int b_lim = (g.N < BN ? g.N : BN) - 1;
    uint32_t voff[LPW];
#pragma unroll
    for (int j = 1; j < LPW; ++j) {
        const int R = 8 * (4 * j + wave) + r_lane;
        const int kc = (lane & 7) ^ ((R >> 1) & 7);
        const int r = min((R - BM) % BN, b_lim);
        voff[j] = static_cast<uint32_t>(r) * static_cast<uint32_t>(4 * g.K) + static_cast<uint32_t>(kc * 16);
    }
    const int ra = min(8 * wave + r_lane, a_lim);  // this lane's activation row in load 0
    const uint32_t kca = static_cast<uint32_t>(((lane & 7) ^ (((8 * wave + r_lane) >> 1) & 7)) * 16);

    // ---- load cursor: work item li, K step lk, scalar bases of the item's rows
    int li = t_first, lk = 0;
    const unsigned char *src_a = nullptr, *src_b0 = nullptr, *src_b1 = nullptr;
    TileGeom lg;  // of the item being loaded
    auto set_item = [&](int L) {
        lg = tile_geom<BM, BN>(g, tiles, L / ks);
        const TileGeom& t = lg;
        const int64_t k0 = static_cast<int64_t>(L % ks) * nk * kF2BK;  // first K value of the item
        if (g.gather) {
            // absolute source row (T h 4 < 4 GiB is checked by the host)
            const int64_t src = source_row(g, row_base<BM>(g, t) + ra);
            voff[0] = static_cast<uint32_t>(src) * static_cast<uint32_t>(4 * g.K) + kca;
            src_a = uniform_ptr(static_cast<const float*>(g.a) + k0);
        } else {
            voff[0] = static_cast<uint32_t>(ra) * static_cast<uint32_t>(4 * g.K) + kca;
            src_a = uniform_ptr(static_cast<const float*>(g.a) + static_cast<int64_t>(row_base<BM>(g, t)) * g.K + k0);
        }
        const int64_t boff = t.e * g.b_estride + static_cast<int64_t>(n_base<BN>(g, t)) * g.K + k0;
        src_b0 = uniform_ptr(static_cast<const float*>(g.b) + boff);
        src_b1 = NB > 1 ? uniform_ptr(static_cast<const float*>(g.b2) + boff) : src_b0;
    };
    int issued = 0;  // stages issued by this wave so far
    auto issue_next = [&]() {
        if (li >= t_end) return;
        const uint32_t dst = lds0 + (issued % NS) * kStageBytes;
        const int kb = lk * kF2BK * 4;  // bytes into every row
#pragma unroll
        for (int j = 0; j < LPW; ++j) {
            const unsigned char* base = j == 0 ? src_a : ((j - 1) / 4 == 0 ? src_b0 : src_b1);
            load_lds16(base + kb, voff[j], dst + (4 * j + wave) * 1024);
        }
        ++issued;
        if (++lk == nk) {
            lk = 0;
            li += nslot;
            if (li < t_end) set_item(li);
        }
    };
    set_item(li);
#pragma unroll
    for (int st = 0; st < NS - 1; ++st) issue_next();

    const int l32 = lane & 31, lhi = lane >> 5;
    // byte offsets of this lane's fragments in a stage
    int xoff[kF2BK / 8], woff[kF2BK / 8];
#pragma unroll
    for (int q = 0; q < kF2BK / 8; ++q) {
        const int slot = 2 * q + lhi, Rw = BM + 32 * wave + l32;
        xoff[q] = l32 * 128 + ((slot ^ ((l32 >> 1) & 7)) << 4);
        woff[q] = Rw * 128 + ((slot ^ ((Rw >> 1) & 7)) << 4);
    }
    int consumed = 0;
    for (int L = t_first; L < t_end; L += nslot) {
        const TileGeom t = nk >= NS ? lg : tile_geom<BM, BN>(g, tiles, L / ks);  // as in gemm_bf16_lds
        f32x16_t acc[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nb][r] = 0.f;

        // publish the item's first stage (after an epilogue its stores share the counter)
        wait_lgkm0();
        if (L != t_first) wait_vmcnt<0>();
        else wait_stages<LPW, NS>(issued - consumed - 1);
        stage_barrier();
        issue_next();
        for (int ck = 0; ck < nk; ++ck) {
            const unsigned char* st = smem_raw + (consumed % NS) * kStageBytes;
#pragma unroll
            for (int q = 0; q < kF2BK / 8; ++q) {
                const float4 xf = *reinterpret_cast<const float4*>(st + xoff[q]);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    // the next matrix's rows are BN further: the same swizzle
                    const float4 wf = *reinterpret_cast<const float4*>(st + woff[q] + nb * BN * 128);
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(wf.x, xf.x, acc[nb], 0, 0, 0);
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(wf.y, xf.y, acc[nb], 0, 0, 0);
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(wf.z, xf.z, acc[nb], 0, 0, 0);
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(wf.w, xf.w, acc[nb], 0, 0, 0);
                }
            }
            ++consumed;
            if (ck + 1 < nk) {
                // publish the next stage: own reads of this one done, own loads of the next
                // landed; then refill this stage's buffer
                wait_lgkm0();
                wait_stages<LPW, NS>(issued - consumed - 1);
                stage_barrier();
                issue_next();
            }
        }

        // ---- epilogue.  Lane: activation row row_base + l32; register 4 q + c: output column
        // n_base + 32 wave + 8 q + 4 lhi + c.
        const int64_t row = row_base<BM>(g, t) + l32;
        const bool row_ok = row >= max(t.row0, 0) && row < t.row_end;
        const int cb = n_base<BN>(g, t) + 32 * wave + 4 * lhi;
        if (ks > 1) {
            // a K part: its fp32 sums go to partial[part][row][N], the reduce kernel finishes
            float* const dst = g.partial + static_cast<int64_t>(L % ks) * g.rows_max * g.N;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = cb + 8 * q;
                if (row_ok && col >= t.n0 && col < g.N)
                    *reinterpret_cast<float4*>(dst + row * g.N + col) =
                        make_float4(acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]);
            }
            continue;
        }
        int64_t orow = row;
        float scale = 1.f;
        if (!kUp && g.scatter) {
            // the grouped row's token and gate weight
            const int64_t src = row_ok ? g.scatter[row] : 0;
            orow = src < 0 ? 0 : (src >= g.c_rows ? g.c_rows - 1 : src);
            scale = row_ok ? g.scatter_w[orow] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int col = cb + 8 * q;
            if (!row_ok || col < t.n0 || col >= g.N) continue;
            float v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = scale * epilogue<EPI>(acc[0][4 * q + c], acc[NB - 1][4 * q + c]);
            if constexpr (OB) {
                uint2 pk;
                pk.x = pack_bf16x2(v[0], v[1]);
                pk.y = pack_bf16x2(v[2], v[3]);
                *reinterpret_cast<uint2*>(static_cast<bf16_t*>(g.c) + orow * g.ldc + col) = pk;
            } else {
                *reinterpret_cast<float4*>(static_cast<float*>(g.c) + orow * g.ldc + col) =
                    make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    }
}

// ------------------------------------------------------------------ few rows per expert: weights streamed into registers
//
// For calls whose experts have few rows (which calls: stream_rows in shapes.h), where reading the
// weights is all the time there is.  A workgroup owns NC weight rows (SwiGLU: NC / 2 of each
// matrix) and a tile of at most 16 MR activation rows of one expert; its NW waves cut K
// between them, so that even one expert's matrix keeps hundreds of waves loading.  A wave
// loads fragments of v_mfma_f32_16x16x32_bf16 (fp32: of four v_mfma_f32_16x16x4_f32) straight
// from global memory, 64 bytes of every row per K step (lane l: 16-byte chunk l / 16 of row
// l % 16), U steps ahead of the ones it multiplies: no LDS, no barrier and no wait but the
// loads' own until the waves add their sums, in wave order, through LDS.  Each weight is
// loaded by one wave of one workgroup (per row tile); the activations, re-read by every
// workgroup, come from L2.
//
// RAG: K is not a whole number of 64-byte steps (an up-projection on row-major weights): the
// chunks past the end are loaded from the row's last one and replaced by zeros.
template <typename T, int EPI, bool OB, int NC, int MR, bool RAG>
__global__ __launch_bounds__(512, MR == 1 ? 4 : 2) void gemm_stream(GroupedGemm g) {
    constexpr bool kBf = std::is_same<T, bf16_t>::value;
    constexpr bool kUp = EPI != kEpiNone;
    constexpr int ES = sizeof(T), BM = 16 * MR, NW = 8, U = NC == 64 ? 1 : 2;
    constexpr int NB = EPI == kEpiSwiglu ? 2 : 1, BN = NC / NB, NJ = NC / 16;
    static_assert(NJ % NB == 0, "whole 16-row blocks of each matrix");
    constexpr bool w_blocked = kBf && !RAG;  // the packed layout
    constexpr int kLd = NC + 4;              // LDS row stride in floats
    __shared__ __align__(16) float red[NW][16][kLd];

    RegTiles<BM> tiles;
    tiles.build(g.offsets, g.E);
    // contiguous runs of the tile list per XCD
    const int total = tiles.total * g.n_tiles, per = (total + 7) >> 3;
    const int slot = static_cast<int>(blockIdx.x >> 3);
    const int L = static_cast<int>(blockIdx.x & 7) * per + slot;
    if (slot >= per || L >= total) return;
    const TileGeom t = tile_geom<BM, BN>(g, tiles, L);

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, chunk = lane >> 4;
    const int64_t kbytes = static_cast<int64_t>(g.K) * ES;
    const int nst = static_cast<int>((kbytes + 63) / 64);
    const int s0 = static_cast<int>(static_cast<int64_t>(nst) * wave / NW);  // this wave's K steps
    const int s1 = static_cast<int>(static_cast<int64_t>(nst) * (wave + 1) / NW);

    // per-lane byte offsets of the rows from uniform bases
    const uint32_t w_row = w_blocked ? 64u : static_cast<uint32_t>(kbytes);
    const int64_t w_step = w_blocked ? static_cast<int64_t>(g.N) * 64 : 64;
    const unsigned char* wbase[NB];
    {
        const int64_t off = t.e * g.b_estride * ES + static_cast<int64_t>(t.n0) * w_row;
        wbase[0] = uniform_ptr(static_cast<const unsigned char*>(g.b) + off);
        if (NB > 1) wbase[NB - 1] = uniform_ptr(static_cast<const unsigned char*>(g.b2) + off);
    }
    uint32_t woff[NJ / NB];
#pragma unroll
    for (int j = 0; j < NJ / NB; ++j)
        woff[j] = static_cast<uint32_t>(min(16 * j + r16, g.N - 1 - t.n0)) * w_row + (RAG ? 0u : 16u * chunk);
    // activations: row-major x, or H (bf16: K-blocked)
    const bool a_blocked = !kUp && kBf;
    const uint32_t a_row = a_blocked ? 64u : static_cast<uint32_t>(kbytes);
    const int64_t a_step = a_blocked ? g.rows_max * 64 : 64;
    const bool gathered = kUp && g.gather;
    const unsigned char* abase = uniform_ptr(static_cast<const unsigned char*>(g.a) + (gathered ? 0 : static_cast<int64_t>(t.row0) * a_row));
    uint32_t aoff[MR];
    const int valid = min(t.row_end - t.row0, BM);
    if (valid <= 0) return;
#pragma unroll
    for (int m = 0; m < MR; ++m) {
        const int r = min(16 * m + r16, valid - 1);
        aoff[m] = static_cast<uint32_t>(gathered ? source_row(g, t.row0 + r) : r) * a_row + (RAG ? 0u : 16u * chunk);
    }

    struct Stage {
        uint4 w[U][NJ], a[U][MR];
    };
    auto load = [&](Stage& st, int s) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t step = min(s + u, s1 - 1);
            const int64_t at = step * 64 + 16 * chunk;
            const uint32_t c = RAG ? static_cast<uint32_t>(at < kbytes ? at : kbytes - 16) : 0u;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const unsigned char* b = wbase[j / (NJ / NB)] + (RAG ? 0 : step * w_step);
                st.w[u][j] = *reinterpret_cast<const uint4*>(b + (woff[j % (NJ / NB)] + c));
            }
#pragma unroll
            for (int m = 0; m < MR; ++m)
                st.a[u][m] = *reinterpret_cast<const uint4*>(abase + (RAG ? 0 : step * a_step) + (aoff[m] + c));
            if (RAG && at >= kbytes) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) st.w[u][j] = make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int m = 0; m < MR; ++m) st.a[u][m] = make_uint4(0, 0, 0, 0);
            }
        }
    };
    f32x4_t acc[NJ][MR];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int m = 0; m < MR; ++m) acc[j][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](const Stage& st, int s) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s + u >= s1) break;
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int m = 0; m < MR; ++m) {
                    if constexpr (kBf) {
                        acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(st.w[u][j]), as_bf16x8(st.a[u][m]),
                                                                            acc[j][m], 0, 0, 0);
                    } else {
                        const float4 w = __builtin_bit_cast(float4, st.w[u][j]), a = __builtin_bit_cast(float4, st.a[u][m]);
                        acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, a.x, acc[j][m], 0, 0, 0);
                        acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.y, a.y, acc[j][m], 0, 0, 0);
                        acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.z, a.z, acc[j][m], 0, 0, 0);
                        acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.w, a.w, acc[j][m], 0, 0, 0);
                    }
                }
        }
    };
    if (s0 < s1) {
        Stage e, o;
        load(e, s0);
        for (int s = s0; s < s1; s += 2 * U) {
            if (s + U < s1) load(o, s + U);
            mma(e, s);
            if (s + 2 * U < s1) load(e, s + 2 * U);
            if (s + U < s1) mma(o, s + U);
        }
    }

    // the waves' sums of 16 rows at a time meet in LDS (D: lane l holds row l % 16, columns
    // 4 (l / 16) .. + 3 of each 16 x 16 block); each thread then owns pairs of columns
#pragma unroll
    for (int m = 0; m < MR; ++m) {
        if (m && 16 * m >= valid) break;
        if (m) __syncthreads();
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            *reinterpret_cast<f32x4_t*>(&red[wave][r16][16 * j + 4 * chunk]) = acc[j][m];
        __syncthreads();
        for (int i = threadIdx.x; i < 16 * BN / 2; i += 64 * NW) {
            const int r = i / (BN / 2), c = (i - r * (BN / 2)) * 2;
            float2 v = *reinterpret_cast<const float2*>(&red[0][r][c]), q = v;
            if (NB > 1) q = *reinterpret_cast<const float2*>(&red[0][r][BN + c]);
#pragma unroll
            for (int w = 1; w < NW; ++w) {
                const float2 b = *reinterpret_cast<const float2*>(&red[w][r][c]);
                v.x += b.x;
                v.y += b.y;
                if (NB > 1) {
                    const float2 d = *reinterpret_cast<const float2*>(&red[w][r][BN + c]);
                    q.x += d.x;
                    q.y += d.y;
                }
            }
            const int n = t.n0 + c;
            if (16 * m + r >= valid || n >= g.N) continue;
            int64_t row = static_cast<int64_t>(t.row0) + 16 * m + r;
            if (!kUp && g.partial) {  // whole sums in fp32, for split_combine
                *reinterpret_cast<float2*>(g.partial + row * g.N + n) = v;
                continue;
            }
            float scale = 1.f;
            if (!kUp && g.scatter) {
                const int64_t src = g.scatter[row];
                row = src < 0 ? 0 : (src >= g.c_rows ? g.c_rows - 1 : src);
                scale = g.scatter_w[row];
            }
            if (kBf) {
                v.x = epilogue_bf16<EPI, RAG>(v.x, q.x);
                v.y = epilogue_bf16<EPI, RAG>(v.y, q.y);
            } else {
                v.x = epilogue<EPI>(v.x, q.x);
                v.y = epilogue<EPI>(v.y, q.y);
            }
            if (!kUp) {
                v.x *= scale;
                v.y *= scale;
            }
            if (kUp && kBf) {
                bf16_t* const d = static_cast<bf16_t*>(g.c) + ((static_cast<int64_t>(n) >> 5) * g.rows_max + row) * 32 + (n & 31);
                *reinterpret_cast<uint32_t*>(d) = pack_bf16x2(v.x, v.y);
            } else if (OB) {
                *reinterpret_cast<uint32_t*>(static_cast<bf16_t*>(g.c) + row * g.ldc + n) = pack_bf16x2(v.x, v.y);
            } else {
                *reinterpret_cast<float2*>(static_cast<float*>(g.c) + row * g.ldc + n) = v;
            }
        }
    }
}

// ------------------------------------------------------------------ split-K reduce
//
// out[p] = sum over s of partial[s][p] (s ascending) for the grouped rows p of the call,
// [offsets[0], offsets[E]); with scatter (top-1), out[t] = w[t] * that sum for
// t = scatter[p] instead (the down-projection's own epilogue, applied after the parts
// meet).  N % 4 == 0.  S (four parts) is a template argument so that a thread's S loads are
// issued together (one memory round trip) before the sum.

template <bool OB, int S>
__global__ __launch_bounds__(256) void split_reduce(const float* __restrict__ partial, int64_t rows_max,
                                                     int N, const int32_t* __restrict__ offsets, int E,
                                                     void* __restrict__ out, int ldo,
                                                     const int32_t* __restrict__ scatter,
                                                     const float* __restrict__ scatter_w, int64_t c_rows) {
    const int64_t p0 = offsets[0];
    const int64_t p1 = offsets[E] < rows_max ? offsets[E] : rows_max;
    const int nv = N / 4;
    const int64_t n = (p1 - p0) * nv;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * 256) {
        const int64_t p = p0 + i / nv;
        const int c = static_cast<int>(i % nv) * 4;
        float4 u[S];
#pragma unroll
        for (int s = 0; s < S; ++s)
            u[s] = *reinterpret_cast<const float4*>(partial + (static_cast<int64_t>(s) * rows_max + p) * N + c);
        float4 v = u[0];
#pragma unroll
        for (int s = 1; s < S; ++s) {
            v.x += u[s].x;
            v.y += u[s].y;
            v.z += u[s].z;
            v.w += u[s].w;
        }
        int64_t row = p;
        if (scatter) {
            const int64_t t = scatter[p];
            row = t < 0 ? 0 : (t >= c_rows ? c_rows - 1 : t);
            const float w = scatter_w[row];
            v.x *= w;
            v.y *= w;
            v.z *= w;
            v.w *= w;
        }
        if (OB) {
            uint2 pk;
            pk.x = pack_bf16x2(v.x, v.y);
            pk.y = pack_bf16x2(v.z, v.w);
            *reinterpret_cast<uint2*>(static_cast<bf16_t*>(out) + row * ldo + c) = pk;
        } else {
            *reinterpret_cast<float4*>(static_cast<float*>(out) + row * ldo + c) = v;
        }
    }
}


// Steps 4 and 5 together for decode-sized calls (hands_over_sums): for token t and 8 columns,
//     y[t] = sum over picks j of w[t, j] * round_ydt(sum over s of partial[s][pos_of[t, j]])
// -- the second product's S parts in order (one where its sums are whole), rounded to y_perm's
// type as the product or split_reduce stores it, then combine's weighted sum (fp32, pick order,
// invalid picks skipped) rounded once: the same bits as the two launches, without writing or
// reading y_perm.
template <bool YB, bool OB, int S>
__global__ __launch_bounds__(256) void split_combine(const float* __restrict__ partial, int64_t rows_max,
                                                     int h, const int32_t* __restrict__ pos_of,
                                                     const float* __restrict__ w, int64_t T, int k,
                                                     void* __restrict__ y) {
    const int nv = h / 8;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= T * nv) return;
    const int64_t t = i / nv;
    const int c = static_cast<int>(i - t * nv) * 8;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < k; ++j) {
        const int32_t p = pos_of[t * k + j];
        if (p < 0 || p >= T * k) continue;
        const float wt = w[t * k + j];
        const float* src = partial + static_cast<int64_t>(p) * h + c;
        float4 u[S], v[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const float* q = src + static_cast<int64_t>(s) * rows_max * h;
            u[s] = *reinterpret_cast<const float4*>(q);
            v[s] = *reinterpret_cast<const float4*>(q + 4);
        }
        float4 a = u[0], b = v[0];
#pragma unroll
        for (int s = 1; s < S; ++s) {
            a.x += u[s].x;
            a.y += u[s].y;
            a.z += u[s].z;
            a.w += u[s].w;
            b.x += v[s].x;
            b.y += v[s].y;
            b.z += v[s].z;
            b.w += v[s].w;
        }
        float r[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        if (YB) {
            // y_perm's bf16 rounding, as split_reduce stores it and combine reads it back
#pragma unroll
            for (int q = 0; q < 8; q += 2) {
                const uint32_t pk = pack_bf16x2(r[q], r[q + 1]);
                r[q] = __uint_as_float(pk << 16);
                r[q + 1] = __uint_as_float(pk & 0xffff0000u);
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] += wt * r[q];
    }
    if (OB) {
        uint4 q;
        q.x = pack_bf16x2(acc[0], acc[1]);
        q.y = pack_bf16x2(acc[2], acc[3]);
        q.z = pack_bf16x2(acc[4], acc[5]);
        q.w = pack_bf16x2(acc[6], acc[7]);
        *reinterpret_cast<uint4*>(static_cast<bf16_t*>(y) + t * h + c) = q;
    } else {
        float4* o = reinterpret_cast<float4*>(static_cast<float*>(y) + t * h + c);
        o[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        o[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    }
}

// ------------------------------------------------------------------ launch

template <int EPI, bool OB>
hipError_t run_f32_lds(GroupedGemm g, int64_t A_max, hipStream_t s) {
    typedef F32Shape<(EPI == kEpiSwiglu) ? 2 : 1> S;
    constexpr size_t lds = S::kBytes;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f32_lds<EPI, OB>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       static_cast<int>(lds));
    if (attr != hipSuccess) return attr;
    g.n_tiles = static_cast<int>(ceil_div(g.N, kF2BN));
    const int64_t items = row_tile_bound(A_max, g.E, kF2BM) * g.n_tiles * (g.ksplit > 1 ? g.ksplit : 1);
    if (items == 0) return hipSuccess;
    // persistent grid: at most kPerCU workgroups per CU, a multiple of the 8 XCDs
    const int64_t blocks = round_up(std::min<int64_t>(items, S::kPerCU * static_cast<int64_t>(device_cus())), 8);
    hipLaunchKernelGGL((gemm_f32_lds<EPI, OB>), dim3(static_cast<unsigned>(blocks)), dim3(kThreads), lds, s, g);
    return hipGetLastError();
}

template <int EPI, bool OB>
hipError_t run_f32(GroupedGemm g, int64_t A_max, hipStream_t s) {
    if (g.K % kF2BK == 0) return run_f32_lds<EPI, OB>(g, A_max, s);
    g.n_tiles = static_cast<int>(ceil_div(g.N, kFBN));
    const int64_t blocks = row_tile_bound(A_max, g.E, kFBM) * g.n_tiles;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL((gemm_f32<EPI, OB>), dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, s, g);
    return hipGetLastError();
}

template <int BM, int BW, int BK, int NS, int EPI, bool OB, int WN = 2, bool RM = false>
hipError_t run_bf16_lds(GroupedGemm g, int64_t A_max, hipStream_t s) {
    typedef LdsShape<BM, BW, BK, NS, EPI, WN> S;
    constexpr size_t lds = S::kBytes;
    constexpr int per_cu = S::kPerCU;
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&gemm_bf16_lds<BM, BW, BK, NS, EPI, OB, WN, RM>),
        hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (attr != hipSuccess) return attr;
    g.n_tiles = static_cast<int>(ceil_div(g.N, S::kBN));
    const int64_t tiles = row_tile_bound(A_max, g.E, BM) * g.n_tiles;
    if (tiles == 0) return hipSuccess;
    // persistent grid: at most per_cu workgroups per CU, a multiple of the 8 XCDs
    const int64_t blocks = round_up(std::min<int64_t>(tiles, static_cast<int64_t>(per_cu) * device_cus()), 8);
    hipLaunchKernelGGL((gemm_bf16_lds<BM, BW, BK, NS, EPI, OB, WN, RM>), dim3(static_cast<unsigned>(blocks)),
                       dim3(S::kThreadsWG), lds, s, g);
    return hipGetLastError();
}

template <int EPI>
hipError_t run_up_pairs(GroupedGemm g, int64_t A_max, hipStream_t s) {
    static const hipError_t attr =
        hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_up_pairs<EPI>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kUpPairBytes));
    if (attr != hipSuccess) return attr;
    g.n_tiles = static_cast<int>(ceil_div(g.N, LdsShape<128, 256, 32, 3, EPI>::kBN));
    const int64_t tiles = row_tile_bound(A_max, g.E, 128) * g.n_tiles;
    if (tiles == 0) return hipSuccess;
    const int64_t blocks = round_up(std::min<int64_t>(tiles, 2 * static_cast<int64_t>(device_cus())), 8);
    hipLaunchKernelGGL((gemm_up_pairs<EPI>), dim3(static_cast<unsigned>(blocks)), dim3(kThreads), kUpPairBytes, s,
                       g);
    return hipGetLastError();
}

template <int EPI, bool OB>
hipError_t run_turns(GroupedGemm g, int64_t A_max, hipStream_t s) {
    static const hipError_t attr =
        hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_turns<EPI, OB>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kTurnBytes));
    if (attr != hipSuccess) return attr;
    g.n_tiles = static_cast<int>(ceil_div(g.N, EPI == kEpiSwiglu ? 128 : 256));
    const int64_t tiles = row_tile_bound(A_max, g.E, 256) * g.n_tiles;
    if (tiles == 0) return hipSuccess;
    const int64_t blocks = round_up(std::min<int64_t>(tiles, device_cus()), 8);
    hipLaunchKernelGGL((gemm_turns<EPI, OB>), dim3(static_cast<unsigned>(blocks)), dim3(512), kTurnBytes, s, g);
    return hipGetLastError();
}

template <typename T, int EPI, bool OB, int NC, int MR>
hipError_t run_stream_t(GroupedGemm g, int64_t A_max, hipStream_t s) {
    g.n_tiles = static_cast<int>(ceil_div(g.N, EPI == kEpiSwiglu ? NC / 2 : NC));
    const int64_t items = row_tile_bound(A_max, g.E, 16 * MR) * g.n_tiles;
    if (items == 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>(round_up(items, 8)));
    if (static_cast<int64_t>(g.K) * sizeof(T) % 64 == 0) {
        hipLaunchKernelGGL((gemm_stream<T, EPI, OB, NC, MR, false>), grid, dim3(512), 0, s, g);
        return hipGetLastError();
    }
    if constexpr (EPI != kEpiNone) {  // the down-projection's K is a multiple of 128
        hipLaunchKernelGGL((gemm_stream<T, EPI, OB, NC, MR, true>), grid, dim3(512), 0, s, g);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

template <typename T, int EPI, bool OB>
hipError_t run_stream(GroupedGemm g, int64_t A_max, hipStream_t s) {
    constexpr bool kDual = EPI == kEpiSwiglu, kBf = std::is_same<T, bf16_t>::value;
    const int nc = stream_width(A_max, g.E, g.N, kDual, device_cus());
    if constexpr (!kDual) {
        if (nc == 16) return run_stream_t<T, EPI, OB, 16, 1>(g, A_max, s);
    }
    if (nc == 32) return run_stream_t<T, EPI, OB, 32, 1>(g, A_max, s);
    if constexpr (kBf) {
        const int blocks = stream_launch_blocks(A_max, g.E, ceil_div(g.N, kDual ? 32 : 64), kBf, device_cus());
        if (blocks == 3) return run_stream_t<T, EPI, OB, 64, 3>(g, A_max, s);
        if (blocks == 2) return run_stream_t<T, EPI, OB, 64, 2>(g, A_max, s);
    }
    return run_stream_t<T, EPI, OB, 64, 1>(g, A_max, s);
}

// An up-projection's tiles on K-blocked weights, or on row-major ones.
template <int BM, int BW, int NS, int EPI>
hipError_t run_bf16_up(GroupedGemm g, int64_t A_max, hipStream_t s) {
    if (g.K % 32 == 0) return run_bf16_lds<BM, BW, 32, NS, EPI, true>(g, A_max, s);
    return run_bf16_lds<BM, BW, 32, NS, EPI, true, 2, true>(g, A_max, s);
}

template <int EPI, bool OB>
hipError_t run_bf16_best(GroupedGemm g, int64_t A_max, hipStream_t s) {
    if constexpr (EPI != kEpiNone) {
        static_assert(OB, "H is bf16");
        switch (up_shape(A_max, g.E, g.K, g.N, EPI == kEpiSwiglu, device_cus())) {
            case kTurns256x256: return run_turns<EPI, OB>(g, A_max, s);
            case kTile64x256: return run_bf16_up<64, 256, 3, EPI>(g, A_max, s);
            case kTile64x128: return run_bf16_up<64, 128, 3, EPI>(g, A_max, s);
            case kTile128x128: return run_bf16_up<128, 128, 4, EPI>(g, A_max, s);
            case kPairs128x256: return run_up_pairs<EPI>(g, A_max, s);
            case kTile128x256: return run_bf16_up<128, 256, 3, EPI>(g, A_max, s);
            default: return hipErrorInvalidValue;
        }
    } else {
        if (g.K % 32 != 0) return hipErrorInvalidValue;  // not reachable through the C ABI (fp % 128 == 0)
        switch (down_shape(A_max, g.E, g.K, g.N, device_cus())) {
            case kTurns256x256: return run_turns<EPI, OB>(g, A_max, s);
            case kTile64x256: return run_bf16_lds<64, 256, 32, 3, EPI, OB>(g, A_max, s);
            case kTile128x128: return run_bf16_lds<128, 128, 32, 4, EPI, OB>(g, A_max, s);
            case kTile128x384: return run_bf16_lds<128, 384, 32, 3, EPI, OB, 4>(g, A_max, s);
            case kTile128x256: return run_bf16_lds<128, 256, 32, 3, EPI, OB>(g, A_max, s);
            default: return hipErrorInvalidValue;
        }
    }
}

template <int EPI>
hipError_t gemm1(bool bf16, bool stream, GroupedGemm g, int64_t A_max, hipStream_t s) {
    if (stream) return bf16 ? run_stream<bf16_t, EPI, true>(g, A_max, s) : run_stream<float, EPI, false>(g, A_max, s);
    return bf16 ? run_bf16_best<EPI, true>(g, A_max, s) : run_f32<EPI, false>(g, A_max, s);
}

// Step 5 folded into the expert step (CombineArgs given, a call that hands_over_sums): the second
// product's fp32 sums go straight into y through split_combine instead of into y_perm.
struct CombineArgs {
    const int32_t* pos_of;
    const float* w;
    int64_t T;
    int k;
    void* y;
    bool y_bf16;
};

template <bool OB, int S>
hipError_t launch_split_reduce_t(const float* partial, int64_t rows_max, int h, int64_t grid_rows,
                                 const int32_t* offsets, int E, void* out, const int32_t* scatter,
                                 const float* scatter_w, int64_t c_rows, hipStream_t s) {
    const int64_t n4 = grid_rows * (h / 4);
    const int blocks = static_cast<int>(std::min<int64_t>(ceil_div(n4, 256), 8LL * device_cus()));
    hipLaunchKernelGGL((split_reduce<OB, S>), dim3(blocks), dim3(256), 0, s, partial, rows_max, h, offsets, E, out, h,
                       scatter, scatter_w, c_rows);
    return hipGetLastError();
}

// four parts: the fp32 down-projection's (down_parts)
hipError_t launch_split_reduce(bool ob, const float* partial, int64_t rows_max, int h, int64_t grid_rows,
                               const int32_t* offsets, int E, void* out, const int32_t* scatter,
                               const float* scatter_w, int64_t c_rows, hipStream_t s) {
    return ob ? launch_split_reduce_t<true, 4>(partial, rows_max, h, grid_rows, offsets, E, out, scatter, scatter_w, c_rows, s)
              : launch_split_reduce_t<false, 4>(partial, rows_max, h, grid_rows, offsets, E, out, scatter, scatter_w, c_rows, s);
}

template <bool YB, bool OB, int S>
hipError_t launch_split_combine_t(const float* partial, int64_t rows_max, int h, const CombineArgs& c, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>(ceil_div(c.T * (h / 8), 256)));
    hipLaunchKernelGGL((split_combine<YB, OB, S>), grid, dim3(256), 0, s, partial, rows_max, h, c.pos_of, c.w, c.T,
                       c.k, c.y);
    return hipGetLastError();
}

hipError_t launch_split_combine(bool yb, int S, const float* partial, int64_t rows_max, int h, const CombineArgs& c,
                                hipStream_t s) {
#define MOE_SPLIT_COMBINE(YBV, OBV)                                                              \
    do {                                                                                       \
        if (S == 1) return launch_split_combine_t<YBV, OBV, 1>(partial, rows_max, h, c, s);   \
        if (S == 4) return launch_split_combine_t<YBV, OBV, 4>(partial, rows_max, h, c, s);   \
    } while (0)
    if (yb && c.y_bf16) MOE_SPLIT_COMBINE(true, true);
    else if (yb) MOE_SPLIT_COMBINE(true, false);
    else if (c.y_bf16) MOE_SPLIT_COMBINE(false, true);
    else MOE_SPLIT_COMBINE(false, false);
#undef MOE_SPLIT_COMBINE
    return hipErrorInvalidValue;
}

// Both matmuls of the expert step.  grid_rows sizes the launches (an upper bound of the
// rows the offsets describe); rows_max is the row count of x_perm, H and y_perm.
hipError_t ffn_pair(const void* x_perm, const int32_t* offsets, int64_t grid_rows, int64_t rows_max, int E,
                    int h, int64_t fp, int act, bool bf16, const void* w1t, const void* w3t, const void* w2t,
                    void* y_perm, bool y_bf16, void* hbuf, hipStream_t s, const int32_t* gather = nullptr,
                    int64_t a_rows = 0, const float* scatter_w = nullptr, const CombineArgs* comb = nullptr,
                    int call_E = 0) {
    if (grid_rows == 0) return hipSuccess;
    // call_E: the call's experts where this launch covers one of them
    const bool stream = stream_rows(rows_max, call_E ? call_E : E, h, fp, act == MOE_ACT_SWIGLU, bf16, device_cus());
    GroupedGemm g1{};
    g1.a = x_perm;
    g1.gather = gather;
    g1.a_rows = a_rows;
    g1.b = w1t;
    g1.b2 = w3t;
    g1.c = hbuf;
    g1.offsets = offsets;
    g1.E = E;
    g1.K = h;
    g1.N = static_cast<int>(fp);
    g1.ldc = static_cast<int>(fp);
    g1.b_estride = fp * h;
    g1.rows_max = rows_max;
    hipError_t err;
    if (act == MOE_ACT_SWIGLU) err = gemm1<kEpiSwiglu>(bf16, stream, g1, grid_rows, s);
    else if (act == MOE_ACT_GELU_TANH) err = gemm1<kEpiGeluTanh>(bf16, stream, g1, grid_rows, s);
    else err = gemm1<kEpiGelu>(bf16, stream, g1, grid_rows, s);
    if (err != hipSuccess) return err;

    GroupedGemm g2{};
    g2.a = hbuf;
    g2.b = w2t;
    g2.b2 = nullptr;
    g2.c = y_perm;
    g2.offsets = offsets;
    g2.E = E;
    g2.K = static_cast<int>(fp);
    g2.N = h;
    g2.ldc = h;
    g2.b_estride = static_cast<int64_t>(h) * fp;
    g2.rows_max = rows_max;
    if (scatter_w) {
        g2.scatter = gather;
        g2.scatter_w = scatter_w;
        g2.c_rows = a_rows;
    }
    // fp32 sums after H in the workspace: parts x rows_max x h
    float* const partial = reinterpret_cast<float*>(static_cast<unsigned char*>(hbuf) +
                                                    round_up(rows_max * fp * (bf16 ? 2 : 4), 256));
    // the parts are chosen from rows_max (the call's row bound), so a per-expert launch of this
    // call splits like the grouped one
    const int parts = down_parts(rows_max, fp, bf16, stream);
    if (comb || parts > 1) {
        g2.ksplit = parts;
        g2.partial = partial;
        if (bf16 && !stream) g2.c = partial;  // whole sums as the tiled kernels' fp32 output
        if (stream) err = bf16 ? run_stream<bf16_t, kEpiNone, false>(g2, grid_rows, s) : run_stream<float, kEpiNone, false>(g2, grid_rows, s);
        else err = bf16 ? run_bf16_best<kEpiNone, false>(g2, grid_rows, s) : run_f32<kEpiNone, false>(g2, grid_rows, s);
        if (err != hipSuccess) return err;
        if (!comb)
            return launch_split_reduce(y_bf16, partial, rows_max, h, grid_rows, offsets, E, y_perm, g2.scatter,
                                       g2.scatter_w, g2.c_rows, s);
        return comb->T == 0 ? hipSuccess : launch_split_combine(y_bf16, parts, partial, rows_max, h, *comb, s);
    }
    if (stream) {
        if (bf16) return y_bf16 ? run_stream<bf16_t, kEpiNone, true>(g2, grid_rows, s) : run_stream<bf16_t, kEpiNone, false>(g2, grid_rows, s);
        return y_bf16 ? run_stream<float, kEpiNone, true>(g2, grid_rows, s) : run_stream<float, kEpiNone, false>(g2, grid_rows, s);
    }
    if (bf16) return y_bf16 ? run_bf16_best<kEpiNone, true>(g2, grid_rows, s) : run_bf16_best<kEpiNone, false>(g2, grid_rows, s);
    return y_bf16 ? run_f32<kEpiNone, true>(g2, grid_rows, s) : run_f32<kEpiNone, false>(g2, grid_rows, s);
}

}  // namespace

hipError_t launch_ffn(const void* x_perm, const int32_t* offsets, int64_t A_max, int E, int h,
                      int64_t fp, int act, bool bf16, const void* w1t, const void* w3t,
                      const void* w2t, void* y_perm, bool y_bf16, void* hbuf, hipStream_t s) {
    return ffn_pair(x_perm, offsets, A_max, A_max, E, h, fp, act, bf16, w1t, w3t, w2t, y_perm, y_bf16, hbuf, s);
}

hipError_t launch_ffn_gather(const void* x, int64_t T, const int32_t* row_src, const int32_t* offsets, int64_t A_max,
                             int E, int h, int64_t fp, int act, bool bf16, const void* w1t, const void* w3t,
                             const void* w2t, void* y_perm, bool y_bf16, void* hbuf, hipStream_t s) {
    return ffn_pair(x, offsets, A_max, A_max, E, h, fp, act, bf16, w1t, w3t, w2t, y_perm, y_bf16, hbuf, s, row_src, T);
}

hipError_t launch_ffn_gather_combine(const void* x, int64_t T, const int32_t* row_src, const int32_t* offsets, int k,
                                     int E, int h, int64_t fp, int act, bool bf16, const void* w1t, const void* w3t,
                                     const void* w2t, void* y_perm, bool y_bf16, const int32_t* pos_of,
                                     const float* topk_w, void* y, bool out_bf16, void* hbuf, hipStream_t s,
                                     bool* y_perm_written) {
    const int64_t A_max = T * k;
    const bool sums = hands_over_sums(A_max, fp, bf16);
    *y_perm_written = !sums;
    if (sums) {
        const CombineArgs comb{pos_of, topk_w, T, k, y, out_bf16};
        return ffn_pair(x, offsets, A_max, A_max, E, h, fp, act, bf16, w1t, w3t, w2t, y_perm, y_bf16, hbuf, s,
                        row_src, T, nullptr, &comb);
    }
    const hipError_t err =
        ffn_pair(x, offsets, A_max, A_max, E, h, fp, act, bf16, w1t, w3t, w2t, y_perm, y_bf16, hbuf, s, row_src, T);
    if (err != hipSuccess) return err;
    return launch_combine(y_perm, y_bf16, pos_of, topk_w, T, k, h, y, out_bf16, s);
}

// One expert at a time: expert e's segment is the one-expert grouping (offsets + e), its
// weights start e matrices into each packed block, and the launches are sized by its own
// row count, read from the host copy of the offsets.
// Top-1 layer output in one call: gathered rows in, y[t] = w[t] * FFN(x[t]) out.
hipError_t launch_ffn_top1(const void* x, int64_t T, const int32_t* row_src, const float* topk_w,
                           const int32_t* offsets, int64_t A_max, int E, int h, int64_t fp, int act, bool bf16,
                           const void* w1t, const void* w3t, const void* w2t, void* y, bool y_bf16, void* hbuf,
                           hipStream_t s) {
    return ffn_pair(x, offsets, A_max, A_max, E, h, fp, act, bf16, w1t, w3t, w2t, y, y_bf16, hbuf, s, row_src, T,
                    topk_w);
}

// ------------------------------------------------------------------ no-allocation variant
//
// The workspace of one call (H, then a small call's fp32 sums) lives in a
// static device array instead of caller memory.  Each GPU the library runs on holds its own
// copy of the array for the life of the process.  In host code the array's name only stands
// in for it: the device address comes from hipGetSymbolAddress, taken once per device with
// that device current, and only that address is ever handed to a kernel.  Nothing in the
// array needs to start at zero (every H row and fp32 sum a kernel reads is written
// earlier in the same call; rows of a tile past its segment only feed outputs that are not
// stored).  Calls that overlap on one GPU share the array and race.
namespace {

__device__ __align__(256) unsigned char scratch[MOE_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxScratchDevices] = {};

// Device address of `scratch` on the current device (resolved on the first call there).
hipError_t static_scratch(void** out) {
    int dev = -1;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess) return err;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace

hipError_t launch_ffn_noalloc(const void* x_perm, const int32_t* offsets, int64_t A_max, int E, int h, int64_t fp,
                              int act, bool bf16, const void* w1t, const void* w3t, const void* w2t, void* y_perm,
                              bool y_bf16, hipStream_t s) {
    if (s) {  // the stream must belong to the current device, whose copy of the array is used
        int sdev = -1, dev = -1;
        hipError_t err = hipStreamGetDevice(s, &sdev);
        if (err != hipSuccess) return err;
        err = hipGetDevice(&dev);
        if (err != hipSuccess) return err;
        if (sdev != dev) return hipErrorInvalidDevice;
    }
    void* ws = nullptr;
    const hipError_t err = static_scratch(&ws);
    if (err != hipSuccess) return err;
    return ffn_pair(x_perm, offsets, A_max, A_max, E, h, fp, act, bf16, w1t, w3t, w2t, y_perm, y_bf16, ws, s);
}

hipError_t launch_ffn_per_expert(const void* x_perm, const int32_t* offsets, const int32_t* offsets_host,
                                 int64_t A_max, int E, int h, int64_t fp, int act, bool bf16, const void* w1t,
                                 const void* w3t, const void* w2t, void* y_perm, bool y_bf16, void* hbuf,
                                 hipStream_t s) {
    const int64_t es = bf16 ? 2 : 4;
    const int64_t mat = fp * h * es;  // bytes of one expert's matrix in each packed block
    for (int e = 0; e < E; ++e) {
        const int64_t count = static_cast<int64_t>(offsets_host[e + 1]) - offsets_host[e];
        if (count <= 0) continue;
        const unsigned char* b1 = static_cast<const unsigned char*>(w1t) + e * mat;
        const unsigned char* b3 = w3t ? static_cast<const unsigned char*>(w3t) + e * mat : nullptr;
        const unsigned char* b2 = static_cast<const unsigned char*>(w2t) + e * mat;
        const hipError_t err = ffn_pair(x_perm, offsets + e, count, A_max, 1, h, fp, act, bf16, b1, b3, b2, y_perm,
                                        y_bf16, hbuf, s, nullptr, 0, nullptr, nullptr, E);
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

}  // namespace moe
