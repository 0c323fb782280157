// Which GEMM kernel takes a call and in what passes: plain C++ without HIP, so that a host compiler can check it.
// Every choice leaves a row's sums as they are; these rules decide about time alone.
#pragma once
#include <stdint.h>

// Row tiles per pass of the few-row kernel before short passes: 32 ... 192 rows in steps of 32 take one pass; more rows take
// passes of 160 or 192 rows, whichever needs fewer.
inline int gemm_full_pass(int M) {
    const int tiles = (M + 31) / 32;
    return tiles <= 6 ? tiles : (M + 191) / 192 < (M + 159) / 160 ? 6 : 5;
}

// How the few-row kernel takes M rows: `passes` passes of `mt` row tiles of 32 rows.
struct GemmPass {
    int mt, passes;
    // Weights are loaded with the default cache policy where several passes read them: the passes of an n-block run
    // side by side on one XCD and find them in its L2.  One pass loads them non-temporally, so that they do not evict
    // the activations.  Non-temporal / default, us: QKV of a 1600-wide model, 512 rows 34.1 / 29.5, its attention output,
    // 1152 rows 33.0 / 26.8, its gate/up, 64 rows in two passes 20.7 / 17.4; gate/up of a 1024-wide model, 448 rows
    // 18.7 / 15.4.  No matrix of the widths 512, 1024, 1600 and 2048 is faster with non-temporal loads in several passes.
    bool cached;
};

// Small matrices, whose n-blocks leave more than half of the CUs idle, take shorter passes until 128 work-groups
// run: a work-group's time is its K walk times its row tiles
// (192 rows, K = 512, us, one pass / short passes: gate/up of 1536 channels 17 / 7.3, LM head of 2080 tokens 14.7 / 9.4,
// attention output 10 / 4.7).
inline GemmPass gemm_few_row_pass(int M, int N, int split, int wn) {
    const int tiles = (M + 31) / 32, blocks = (N / 32 + wn - 1) / wn * split;
    int mt = gemm_full_pass(M);
    while (mt > 1 && (long long)blocks * ((tiles + mt - 1) / mt) < 128) --mt;
    const int passes = (tiles + mt - 1) / mt;
    return GemmPass{mt, passes, passes > 1};
}

// The tiles of k_gemm_rows, weight rows x activation rows.  HALVES: tiles that walk one half of the k-slices and add their sums, so that
// two partial sums leave the kernel (fp32 partial sums in more than two slices only).
enum GemmTile {
    GEMM_FEW_ROWS = 0,                                       // not one of them: the few-row kernel
    GEMM_256x96 = 256096, GEMM_256x128 = 256128, GEMM_256x160 = 256160, GEMM_192x256 = 192256, GEMM_192x320 = 192320, GEMM_256x256 = 256256,
    GEMM_HALVES_192x128 = 2192128, GEMM_HALVES_256x128 = 2256128
};

// n-tiles of the few-row kernel's work-groups for gate/up: three where they divide the matrix (the 8B shape, 768 tiles: a work-group on
// every CU), for one row tile, whose loads smaller blocks spread better over the CUs, and for rows of one pass where at least 160 blocks
// remain.  Blocks of four / three, us: 1184 tiles, of which 40 CUs get two blocks of four, 8 rows 56.1 / 46.9, 32 rows 58.4 / 49.1, 192 rows
// 90 / 83; 512 tiles 32 rows 25.3 / 21.9, 192 rows 40.2 / 37.9; 400 tiles 32 rows 15.6 / 14.0, 192 rows 21.3 / 22.9.
inline int gemm_channels_block(int M, int N) {
    const int tiles = N / 32;
    return tiles % 3 == 0 || M <= 32 || (M <= 192 && tiles >= 480) ? 3 : 4;
}

// What a GEMM writes: split-K partial sums, activated channels, the LM head's partial results.
enum GemmOut { GEMM_SUMS, GEMM_CHANNELS, GEMM_LM };

// The kernel for M rows of a matrix with N weight rows and `split` k-slices of nch chunks of 64 columns; wn: n-tiles of the few-row
// kernel's work-groups.  Up to 192 rows the few-row kernel needs one pass over the weights and every CU streams its own share of
// them.  For more rows the way with the least estimated time:
//     rounds over the 256 CUs x (round + chunks x chunk) + share of the chip's work-group slots x chunks x full + weights x w
//     + 0.69 ns per 1000 partial sums, written and read again by the consumer (0.17 us per MB)
// `full` on top of `chunk` because a round that fills the chip only partly draws less power and clocks higher.  Few-row kernel: chunk
// and full grow with the loads (n-tiles + row tiles) and the products (n-tiles x row tiles) of a work-group; several slices cost 12 %
// more, and of the LM head, whose work-groups share a CU in pairs, an even number of passes 8 % less, an odd one 20 % more.
// Fitted to the times of kernel and consumer inside forwards of seven shapes (widths 1024, 1600, 2048, 3072, 3584, 4096 and 5120, five
// matrices each, 193 to 2304 rows, 805 calls with every way each; one way's time is met within 5 to 10 % rms).  The choice is 0.15 %
// slower than the fastest way on average, 0.7 % at the 95th percentile, 8 % at most (rules of their own for the large, the small and the
// halving tiles: 1.4, 8.4 and 21 %); a shape left out of the fit lost 0.1 to 0.4 %.  8B shape, attention output
// and a layer's norms, us, best without halves / halves: 512 rows 55 / 59, 640 rows 54.8 / 54.4, 1000 rows 75 / 72; down 512 rows 79 / 94,
// 640 rows 103 / 100, 1000 rows 143 / 128.
// At least 112 work-groups: with fewer, half of the chip idle, the few-row kernel's narrower n-blocks spread better (120 work-groups, 2560
// wide, attention output and norms at 193 rows: few-row kernel 34.3, 256 x 96 30.9).
inline int gemm_tile(int M, int N, int nch, int split, int wn, GemmOut out) {
    if (M <= 192) return GEMM_FEW_ROWS;
    struct Kind { int code, nt, mt; double round, chunk, full, w; };         // tiles of 32 rows; ns
    static const Kind kinds[8] = {
        {GEMM_256x96, 8, 3, 6663, 446, 132, .161}, {GEMM_256x128, 8, 4, 7910, 463, 232, .142}, {GEMM_256x160, 8, 5, 8614, 489, 369, .110},
        {GEMM_192x256, 6, 8, 9117, 578, 437, .111}, {GEMM_192x320, 6, 10, 9540, 716, 537, .088}, {GEMM_256x256, 8, 8, 10682, 617, 753, .078},
        {GEMM_HALVES_192x128, 6, 4, 7927, 438, 197, .113}, {GEMM_HALVES_256x128, 8, 4, 9289, 559, 260, .064}};
    const double weights = (double)N * nch * split * 64 / 1000, sums = out == GEMM_SUMS ? .69 * M * N / 1000 : 0;
    const GemmPass p = gemm_few_row_pass(M, N, split, wn);
    const long long few_wgs = (long long)((N / 32 + wn - 1) / wn) * split * p.passes;
    int best = GEMM_FEW_ROWS;
    double least = ((few_wgs + 255) / 256 * (4996 + nch * (26.8 * (wn + p.mt) + 10.7 * wn * p.mt)) +
                    few_wgs * nch * 6.9 * wn * p.mt / 256 + weights * .08) *
                       (split > 1 ? 1.12 : out == GEMM_LM && few_wgs > 256 ? (p.passes % 2 ? 1.2 : .92) : 1.03) +
                   split * sums;
    for (const Kind& k : kinds) {
        const bool half = k.code >= GEMM_HALVES_192x128;
        if (half && (out != GEMM_SUMS || split <= 2)) continue;
        const int parts = half ? 2 : split, chunks = half ? nch * ((split + 1) / 2) : nch;
        const long long wgs = (long long)((N / 32 + k.nt - 1) / k.nt) * parts * ((M + k.mt * 32 - 1) / (k.mt * 32));
        const double t = (wgs + 255) / 256 * (k.round + chunks * k.chunk) + wgs * chunks * k.full / 256 + weights * k.w + parts * sums;
        if (wgs >= 112 && t < least) { best = k.code; least = t; }
    }
    return best;
}

// Plain GEMM: k_gemm_plain_small may take the call while k_gemm_plain's 64x64 tiles would give a CU at most one work-group.
// Unaligned operands (kernel-level entry points take any pointer) stay with the scalar loads.
#define GEMM_PLAIN_TILE 64
inline bool gemm_plain_small_tiles(const void* X, const void* W, int M, int N) {
    const long long tiles = (long long)((N + GEMM_PLAIN_TILE - 1) / GEMM_PLAIN_TILE) * ((M + GEMM_PLAIN_TILE - 1) / GEMM_PLAIN_TILE);
    return tiles <= 256 && (((uintptr_t)X | (uintptr_t)W) & 15) == 0;
}

// It does for up to 64 rows, and for more rows up to 160 tiles: its 16 rows share nothing, so every 16 rows read the weights
// again (us, 64x64 tiles / small ones; up to 64 rows: 60 tiles 12.7 / 6.4, 125 tiles 43 / 30, 192 tiles 4096 wide 172 / 106 and 257 /
// 220; more rows: 120 tiles 13.2 / 11.7, 144 tiles 36 / 32, 160 tiles 54 / 45, 176 tiles 40 / 43, 192 tiles 20 / 25, 256
// tiles 40 / 60).
inline bool gemm_plain_small_wins(int M, int N) {
    return M <= 64 || (long long)((N + GEMM_PLAIN_TILE - 1) / GEMM_PLAIN_TILE) * ((M + GEMM_PLAIN_TILE - 1) / GEMM_PLAIN_TILE) <= 160;
}

// Attention: work-groups of four waves, two to a CU, where eight-wave ones would take more than one round over the 256 CUs
// (8B shape, us, eight waves / four: 576 work-groups of 64-row blocks 33.6 / 27.7, 640 at prefix 1152 59 / 48, 1000-row
// prompt 50 / 39, refresh of 512 rows 43 / 31; 160 work-groups 13.2 / 13.0, 32 at prefix 1000 18.2 / 19.0).
inline bool attn_two_per_cu(long long work_groups) { return work_groups > 256; }

// Plain attention, one wave per row and query head: whether a wave takes a SIMD's whole register file for loads in flight.  The 1024
// SIMDs have one wave each up to 1024 waves; two channels per lane (head size 128) hold twice the values, in bf16 at no gain.
// Rotary stage and attention, us, deep / not, prefix 384: head size 64, fp32 1024 waves 34.3 / 39.9, 1536 44.3 / 42.8, 4096 71 / 54,
// bf16 1024 waves 34.5 / 35.8, 1536 46.7 / 38.3; head size 128, fp32 512 waves 35.5 / 38.5, 768 40.1 / 40.7 (prefix 16: 29.4 / 25.6),
// 1024 45 / 42, 5120 122 / 94, bf16 256 waves 45 / 39, 5120 177 / 81.
inline bool attn_plain_deep(long long waves, int head_dim, int element_bytes) {
    return head_dim == 64 ? waves <= 1024 : element_bytes == 4 && waves <= 512;
}
