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

// Row tiles (of 32 rows) per work-group of k_gemm_rows, or 0: the few-row kernel takes the call, in n-blocks of wn tiles.
// Up to 192 rows the few-row kernel needs one pass over the weights and every CU streams its own share of them;
// beyond that it re-streams them per pass (gate/up of the 8B shape, us, few-row against k_gemm_rows: 200 rows 83 / 60,
// 576 rows 150 / 117, 1000 rows 283 / 183).  Fewer than 128 work-groups leave half of the chip idle: then the
// few-row kernel's narrower n-blocks spread better.  Among the tiles the fewest rounds over the 256 CUs win, a
// round of 96, 128 or 160 rows costing 0.78 : 1 : 1.3 (measured at 640 and 1000 rows: 47, 59 and 78 us a
// round; the 160-row tile has registers for one weight chunk in flight only, the others for three).
// The few-row kernel's 96-row n-blocks, where they fill the chip, count along: a round of 160 or 192 rows costs 0.65 or
// 0.75 there.  That keeps it for 321 to 384 rows of the 8B shape: QKV 63.5 - 65.2 us (k_gemm_rows 65.9 - 69.4), gate/up
// 97.6 - 103.8 (99.1 - 105.9), sixteen layers and the LM head at 352 rows 4.46 ms (4.70), at 384 rows 4.57 (4.84).
// Its 128- and 64-row n-blocks are no faster there (down 59.7 - 62.6 / 58.8 - 62.4, attention output 34.5 - 35.8 /
// 24.4 - 26.8).
// X, the activations, must start on 16 bytes (their rows then do: K is a multiple of 64): k_gemm_rows copies them to LDS in
// 16-byte pieces.  The kernel-level entry points take any pointer; the few-row kernel reads others as it always did.
inline int gemm_rows_tile(const void* X, int M, int N, int split, int wn) {
    if (M <= 192 || ((uintptr_t)X & 15)) return 0;
    const int n_blocks = (N / 32 + 7) / 8, cost[3] = {78, 100, 130};
    int best = 0, best_cost = 0;
    for (int mt = 3; mt <= 5; ++mt) {
        const long long wgs = (long long)n_blocks * split * ((M + mt * 32 - 1) / (mt * 32));
        const long long c = (wgs + 255) / 256 * cost[mt - 3];
        if (wgs >= 128 && (best == 0 || c < best_cost)) { best = mt; best_cost = (int)c; }
    }
    const long long blocks = (long long)((N / 32 + wn - 1) / wn) * split;
    if (wn == 3 && blocks >= 256) {
        const int mt = gemm_full_pass(M);
        if ((blocks * ((M + mt * 32 - 1) / (mt * 32)) + 255) / 256 * (mt == 6 ? 75 : 65) < best_cost) return 0;
    }
    return best;
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

// Plain GEMM: k_gemm_plain_small takes the call while k_gemm_plain's 64x64 tiles would give a CU at most one work-group
// (fp32, us, 64x64 tiles / small ones: 12 tiles 51 / 5, 60 tiles 57 / 16, 120 tiles 105 / 35, 165 tiles 68 / 44, 240 tiles
// 105 / 70; bf16, N = 4096, K = 12288: 64 tiles 1271 / 236, 192 tiles 1300 / 639, 256 tiles 1322 / 978; the small ones
// read LDS three times as much per FMA).
// Unaligned operands (kernel-level entry points take any pointer) stay with the scalar loads.
#define GEMM_PLAIN_TILE 64
inline bool gemm_plain_small_tiles(const void* X, const void* W, int M, int N) {
    const long long tiles = (long long)((N + GEMM_PLAIN_TILE - 1) / GEMM_PLAIN_TILE) * ((M + GEMM_PLAIN_TILE - 1) / GEMM_PLAIN_TILE);
    return tiles <= 256 && (((uintptr_t)X | (uintptr_t)W) & 15) == 0;
}
